// Host side of libplora: argument validation, the segment-packing metadata builder, workspace
// layout and the launch sequences of the forward and backward calls.  No arithmetic of the layer
// happens here; every step runs in the HIP kernels.
#include "plora_internal.h"
#include "plora_bench.h"
#include "plora_debug.h"

#include <cmath>
#include <cstring>
#include <algorithm>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

namespace plora {

// Limits that keep every index of every kernel inside the type it is computed in: 32-bit byte offsets inside a
// GEMM tile (255 rows x d x 2 bytes), int tile counts, 65535 workgroups along y in the fp32 kernels.
constexpr int64_t kMaxHidden = 1 << 22;
constexpr int64_t kMaxTiles = 1 << 30;

static plora_status validate(const plora_desc *d)
{
    if (!d) return PLORA_ERR_NULL;
    if (d->dtype != PLORA_BF16 && d->dtype != PLORA_F32) return PLORA_ERR_UNSUPPORTED;
    if (d->w_layout != PLORA_W_IN_OUT && d->w_layout != PLORA_W_OUT_IN) return PLORA_ERR_UNSUPPORTED;
    if (d->T < 0 || d->d_in <= 0 || d->d_out <= 0) return PLORA_ERR_SHAPE;
    if (d->T > INT32_MAX || d->d_in > kMaxHidden || d->d_out > kMaxHidden) return PLORA_ERR_SHAPE;
    if (d->dtype == PLORA_BF16 && (d->d_in % 8 != 0 || d->d_out % 8 != 0)) return PLORA_ERR_SHAPE;
    {
        const int64_t tm = (d->T + kGemmTileRows - 1) / kGemmTileRows;
        const int64_t tn = (std::max(d->d_in, d->d_out) + 255) / 256;
        if (tm * tn > kMaxTiles) return PLORA_ERR_SHAPE;
        if (d->dtype == PLORA_F32 && (d->T + 63) / 64 > 65535) return PLORA_ERR_SHAPE;
    }
    if (d->n_seg < 0 || d->n_seg > PLORA_MAX_SEGMENTS) return PLORA_ERR_SEGMENTS;
    if (d->n_adapters < 0 || d->n_adapters > PLORA_MAX_ADAPTERS) return PLORA_ERR_ADAPTER;
    if (d->n_seg == 0) return d->T == 0 ? PLORA_OK : PLORA_ERR_SEGMENTS;
    if (!d->seg_off || !d->seg_adapter) return PLORA_ERR_NULL;
    if (d->n_adapters > 0 && (!d->rank || !d->scale)) return PLORA_ERR_NULL;
    for (int32_t k = 0; k < d->n_adapters; ++k)
        if (d->rank[k] < 1 || d->rank[k] > PLORA_MAX_RANK) return PLORA_ERR_RANK;
    if (d->seg_off[0] != 0 || d->seg_off[d->n_seg] != d->T) return PLORA_ERR_SEGMENTS;
    for (int32_t s = 0; s < d->n_seg; ++s) {
        if (d->seg_off[s + 1] < d->seg_off[s]) return PLORA_ERR_SEGMENTS;
        if (d->seg_adapter[s] < -1 || d->seg_adapter[s] >= d->n_adapters) return PLORA_ERR_ADAPTER;
    }
    return PLORA_OK;
}

// Compact description of a call (the words the preparation kernel receives).  Pointer tables may be null.
// at_base: device address of the packed-A^T region of the workspace (null when only the layout matters).
static void fill_desc_words(const plora_desc *d, int32_t n_blocks, const void *const *A, const void *const *B,
                            float *const *dA, float *const *dB, const void *at_base, bool order_is_identity, uint32_t *w)
{
    auto put64 = [&](int i, uint64_t v) { w[i] = (uint32_t)v; w[i + 1] = (uint32_t)(v >> 32); };
    put64(0, (uint64_t)d->T); put64(2, (uint64_t)d->d_in); put64(4, (uint64_t)d->d_out);
    w[6] = (uint32_t)d->n_seg; w[7] = (uint32_t)d->n_adapters; w[8] = (uint32_t)n_blocks;
    w[9] = (d->w_layout == PLORA_W_OUT_IN ? 1u : 0u) | (order_is_identity ? 2u : 0u) | (d->dtype == PLORA_BF16 ? 4u : 0u);
    put64(10, (uint64_t)(uintptr_t)at_base);
    uint32_t *p = w + kDescHeadWords;
    for (int32_t s = 0; s < d->n_seg; ++s) { *p++ = (uint32_t)d->seg_off[s + 1]; *p++ = (uint32_t)d->seg_adapter[s]; }
    for (int32_t k = 0; k < d->n_adapters; ++k) {
        const int i = (int)(p - w);
        put64(i + 0, (uint64_t)(uintptr_t)(A ? A[k] : nullptr));
        put64(i + 2, (uint64_t)(uintptr_t)(B ? B[k] : nullptr));
        put64(i + 4, (uint64_t)(uintptr_t)(dA ? dA[k] : nullptr));
        put64(i + 6, (uint64_t)(uintptr_t)(dB ? dB[k] : nullptr));
        w[i + 8] = (uint32_t)d->rank[k];
        std::memcpy(&w[i + 9], &d->scale[k], 4);
        p += kDescAdWords;
    }
}

// Everything the host derives from a description: the tables (same code as the device runs), the
// launch plans and the workspace layout.  Depends on the description only (not on pointers or scales),
// so it is kept in a small cache and shared by the calls that repeat a layout - the seven linears of a
// decoder layer, every layer, forward and backward.
struct HostMeta {
    TableLayout layout;
    std::vector<char> image;          // the tables as the device lays them out (pointer fields null)
    Tables t;
    MetaHeader hdr;
    WorkspaceLayout ws;               // plora_linear_fwd / _bwd
    WorkspaceLayout ws_nf4;           // plora_linear_fwd_nf4 / _bwd_nf4: the same places, but only the partial tiles of their own plans
    WorkspaceLayout ws_lora;          // plora_lora_fwd / _bwd: the padded small-matrix region holds [max(d_in, d_out)][rp]
    size_t h_elems = 0, hb_elems = 0, zt_elems = 0, at_elems = 0, ap_elems = 0;
    int r16_total = 0, n_active = 0, max_rank = 0, split_dA = 1, split_dB = 1;
    int split_shrink = 1, split_dh = 1, skinny_cap = 8;   // skinny_cap: splits whose partial tiles the workspace holds
    int short_cap() const { return skinny_cap > 1 ? skinny_cap / 2 : 1; }     // ... and what one of two short products takes of them
    int slices16 = 0;                 // 16-token slices with tokens of an adapter
    int slices_all = 0;               // the same with those of the base model alone
    size_t fwd_parts = 0;             // forward in two launches (gemm_short_bf16.hip): bytes of the shrink's partial sums, in front of the product's; else 0
    size_t dx_part[2] = {};           // dX in the launch of the weight gradients: where its partial tiles lie; else 0 ([1]: as gemm_dx)
    int mean_r16 = 0;                 // their rank padded to 16, on average over the tokens
    GemmPlan gemm_fwd[2], gemm_dx[2];  // [1]: over a weight that the call itself has expanded
    int n_words = 0;
    bool small_part_is_dB = false;    // which of dB and dA has the smaller set of partial tiles
    bool order_is_identity = false;   // the sorted order of the GEMM row tiles is 0, 1, 2, ...: the device need not sort
};

// Flags of one short product.
static size_t flag_count(const MetaHeader &h) { return (size_t)h.n_blocks * kShortSlices * kShortMaxSplits; }

static void build_meta(const plora_desc *d, HostMeta &m)
{
    int32_t n_blocks = 0;
    for (int32_t s = 0; s < d->n_seg; ++s)
        if (d->seg_adapter[s] >= 0) n_blocks += (d->seg_off[s + 1] - d->seg_off[s] + kSkinnyRows - 1) / kSkinnyRows;
    m.n_words = desc_words(d->n_seg, d->n_adapters);
    std::vector<uint32_t> words((size_t)m.n_words);
    fill_desc_words(d, n_blocks, nullptr, nullptr, nullptr, nullptr, nullptr, false, words.data());
    m.layout = table_layout(d->T, d->n_seg, d->n_adapters, n_blocks, d->dtype == PLORA_BF16);
    m.image.assign(m.layout.bytes, 0);
    m.t = tables_at(m.image.data(), m.layout);
    const DescReader<WordsInMemory> in{WordsInMemory{words.data()}};
    std::vector<int32_t> scratch(2 * (size_t)d->n_adapters + 1);
    derive_tables(in, m.t, scratch.data());
    m.order_is_identity = true;
    for (int64_t i = 0; i < m.layout.n_tiles; ++i) m.order_is_identity = m.order_is_identity && m.t.tile_order[i] == (int32_t)i;
    m.hdr = *m.t.hdr;

    int64_t h = 0, hb = 0, zt = 0, at = 0, ap = 0, rows = 0, row_ranks = 0;
    for (int32_t s = 0; s < d->n_seg; ++s) {
        const SegInfo &g = m.t.seg[s];
        m.slices_all += (g.row1 - g.row0 + 15) / 16;
        if (g.adapter < 0) continue;
        const int64_t len = g.row1 - g.row0;
        h += len * g.r; hb += len * g.rp; zt += (int64_t)g.r16 * g.lp;
        m.slices16 += (int)((len + 15) / 16);
        rows += len; row_ranks += len * g.r16;
    }
    m.mean_r16 = rows > 0 ? (int)((row_ranks + rows - 1) / rows) : 0;
    m.r16_total = 0; m.n_active = 0;
    for (int32_t k = 0; k < d->n_adapters; ++k) {
        const AdapterInfo &a = m.t.ad[k];
        at += (int64_t)a.r16 * d->d_in;
        ap += (int64_t)a.rp * (m.hdr.w_out_in ? d->d_out : d->d_in);
        m.r16_total += a.r16;
        m.max_rank = std::max(m.max_rank, a.r);
        m.n_active += a.tokens > 0;
    }
    m.h_elems = (size_t)h; m.hb_elems = (size_t)hb; m.zt_elems = (size_t)zt;
    m.at_elems = (size_t)at; m.ap_elems = (size_t)ap;
    m.split_dA = tokc_splits(m.hdr, d->d_in, d->d_out, m.n_active);
    m.split_dB = tokc_splits(m.hdr, d->d_out, d->d_in, m.n_active);
    m.split_shrink = skinny_splits(m.hdr, d->d_in);
    m.split_dh = skinny_splits(m.hdr, d->d_out);

    const bool bf = d->dtype == PLORA_BF16;
    int max_ext = 0;
    for (int64_t i = 0; i < m.layout.n_tiles; ++i) max_ext = std::max(max_ext, (int)m.t.tile[i].n_ext);
    const bool w_out_in = m.hdr.w_out_in != 0;
    const bool short_shrink = bf && m.hdr.n_blocks > 0 && m.n_words <= kChunkWords && skinny_is_short(m.hdr, m.slices16, m.r16_total, d->d_in);
    GemmShape fwd_shape[2], dx_shape[2];
    for (int i = 0; i < 2; ++i) {
        fwd_shape[i] = GemmShape{d->T, d->d_in, d->d_out, !w_out_in, i == 1, short_shrink && i == 0, max_ext};
        dx_shape[i] = GemmShape{d->T, d->d_out, d->d_in, w_out_in, i == 1, false, max_ext};
        m.gemm_fwd[i] = gemm_plan(fwd_shape[i]);
        m.gemm_dx[i] = gemm_plan(dx_shape[i]);
    }
    auto split_bytes = [&](const GemmPlan &p, int64_t N) { return p.n_split > 1 ? (size_t)p.n_split * d->T * N * 4 : (size_t)0; };
    auto fwd_bytes = [&]() { return std::max(split_bytes(m.gemm_fwd[0], d->d_out), split_bytes(m.gemm_fwd[1], d->d_out)); };
    auto dx_bytes = [&]() { return std::max(split_bytes(m.gemm_dx[0], d->d_in), split_bytes(m.gemm_dx[1], d->d_in)); };
    int skinny_cap = 8;
    bool packed = bf;                            // A_k and B_k packed: only ever read by tokens with an adapter
    auto lay_out = [&](WorkspaceLayout &w, size_t meta_bytes, size_t ap_elems, bool split_gemm, size_t flag_bytes) {
        size_t o = 0;
        w.zero = o; o += kZeroBytes;
        w.meta_bytes = meta_bytes;
        w.meta = o; o = align_up(o + w.meta_bytes, 256);
        w.desc = o; o = align_up(o + (m.n_words > kChunkWords ? (size_t)m.n_words * 4 : 0), 256);
        w.flags = o; o = align_up(o + flag_bytes, 256);
        w.at = o;   o = align_up(o + (packed ? m.at_elems * 2 : 0), 256);
        w.ap = o;   o = align_up(o + (packed ? ap_elems * 2 : 0), 256);
        w.hb = o;   o = align_up(o + (bf ? m.hb_elems * 2 : 0), 256);
        w.zt_h = o; o = align_up(o + (bf ? m.zt_elems * 2 : 0), 256);
        w.zt_g = o; o = align_up(o + (bf ? m.zt_elems * 2 : 0), 256);
        w.hf = o;   o = align_up(o + m.h_elems * 4, 256);
        w.gf = o;   o = align_up(o + (bf ? 0 : m.h_elems * 4), 256);
        w.part = o; o = align_up(o + (bf ? (size_t)skinny_cap * m.hdr.n_blocks * kSkinnyRows * m.hdr.max_r16 * 4 : 0), 256);
        const size_t a_bytes = m.split_dA > 1 ? (size_t)m.split_dA * m.r16_total * d->d_in * 4 : 0;
        const size_t b_bytes = m.split_dB > 1 ? (size_t)m.split_dB * m.r16_total * d->d_out * 4 : 0;
        w.wpart = o; o = align_up(o + (bf ? (a_bytes > b_bytes ? a_bytes : b_bytes) : 0), 256);
        // the GEMMs run when every other partial tile has been summed: theirs take the same place
        w.gpart = w.part;
        if (bf && split_gemm)
            o = std::max(o, align_up(w.gpart + std::max(fwd_bytes(), dx_bytes()), 256));
        w.total = o + 256;
    };
    // What plora_linear_fwd_noalloc takes: a description that fits its scratch array with eight skinny splits, no split GEMM
    // and the tables without their records and flags.  The workspace of such a description must not outgrow the array; any other
    // workspace is larger than the array, so its size alone tells the two apart.
    const bool any_short = bf && (skinny_is_short(m.hdr, m.slices16, m.r16_total, d->d_in) || skinny_is_short(m.hdr, m.slices16, m.r16_total, d->d_out));
    const size_t flag_bytes = any_short ? 2 * flag_count(m.hdr) * sizeof(unsigned long long) : 0;
    lay_out(m.ws, m.layout.blk, m.ap_elems, false, 0);
    const bool fits_scratch = m.ws.total <= (size_t)PLORA_NOALLOC_SCRATCH_BYTES;
    auto outgrown = [&]() {
        lay_out(m.ws, m.layout.bytes, m.ap_elems, true, flag_bytes);
        return fits_scratch && m.ws.total > (size_t)PLORA_NOALLOC_SCRATCH_BYTES;
    };
    // What sticks out is cut: the split GEMM's partial tiles where they reach furthest, else the skinny ones (the two overlay
    // each other; cutting the one that ends earlier would cost its splits and gain no room: 1228 tokens, 4096 -> 28672, 8
    // adapters of rank 8: shrink and dH keep 16 splits instead of 8), first what they have in reserve.  The records (some
    // 100 bytes per token block and adapter) are less than seven skinny splits of 8 KB and more per token block; without token
    // blocks they are less than the packed matrices, which nothing reads then.
    skinny_cap = std::max(8, std::max(m.split_shrink, m.split_dh));
    while (outgrown()) {
        const size_t fwd = fwd_bytes(), dx = dx_bytes();
        if (align_up(m.ws.gpart + std::max(fwd, dx), 256) + 256 == m.ws.total && fwd + dx > 0) {
            for (int i = 0; i < 2; ++i) {
                GemmPlan &p = (fwd > dx ? m.gemm_fwd : m.gemm_dx)[i];
                if (split_bytes(p, fwd > dx ? d->d_out : d->d_in) < std::max(fwd, dx)) continue;
                // 256 x 256 tiles in fewer parts would leave compute units idle: planned anew, those with less room.  Small tiles are
                // then cut part by part.  Planned within less room as well they would mostly be whole; 24 such steps, us, cut and whole: 3 %
                // for the whole ones on average (880 x 27696 -> 3280 630 and 553, 1304 x 3208 -> 21360 691 and 644), but 498 x 10600 ->
                // 15648 554 and 610, 396 x 15104 -> 10360 472 and 519, 433 x 10016 -> 14096 506 and 549, 758 x 6928 -> 24568 806 and 846
                if (p.bm == 0) p = gemm_plan(fwd > dx ? fwd_shape[i] : dx_shape[i], (double)std::max(fwd, dx) - 1.0);
                else p.n_split -= 1;
            }
        } else if (m.hdr.n_blocks > 0 && skinny_cap > 1) {
            skinny_cap -= 1;
            m.split_shrink = std::min(m.split_shrink, skinny_cap);
            m.split_dh = std::min(m.split_dh, skinny_cap);
        } else if (m.hdr.n_blocks == 0 && packed) {
            packed = false;
        } else {
            break;
        }
    }
    // the dense calls and those on an expanded weight (index 1) have the partial tiles of their own products alone
    lay_out(m.ws, m.layout.bytes, m.ap_elems, false, flag_bytes);
    size_t total[2];
    for (int i = 0; i < 2; ++i)
        total[i] = !bf ? m.ws.total : std::max(m.ws.total, align_up(m.ws.gpart + std::max(split_bytes(m.gemm_fwd[i], d->d_out), split_bytes(m.gemm_dx[i], d->d_in)), 256) + 256);
    packed = bf;
    // dB and dA share a launch: the larger set of their partial tiles has the region of its own, the smaller lies over the
    // skinny ones and is split no further than fits there
    {
        const size_t room = (size_t)skinny_cap * m.hdr.n_blocks * kSkinnyRows * m.hdr.max_r16 * 4;
        auto bytes = [&](int n, int64_t C) { return n > 1 ? (size_t)n * m.r16_total * C * 4 : (size_t)0; };
        m.small_part_is_dB = bytes(m.split_dB, d->d_out) <= bytes(m.split_dA, d->d_in);
        int &n = m.small_part_is_dB ? m.split_dB : m.split_dA;
        while (bytes(n, m.small_part_is_dB ? d->d_out : d->d_in) > room) n -= 1;
    }
    int64_t rp_total = 0;
    for (int32_t k = 0; k < d->n_adapters; ++k) rp_total += m.t.ad[k].rp;
    lay_out(m.ws_lora, m.layout.bytes, (size_t)(rp_total * std::max(d->d_in, d->d_out)), false, flag_bytes);
    m.skinny_cap = skinny_cap;
    // Forward in two launches: where the shrink is short and the base product is split anyway, or its one set of fp32 sums costs less
    // than the launch saved.  Both ways at 84 unsplit products, time in two launches over that in three: up to 1.4 M sums 0.78 to 0.79, 1.4 - 1.9 M
    // 0.75 to 0.93, 1.9 - 2.4 M 0.70 to 1.01 (2020 x 968 -> 1080 26.6 and 26.9 us), 2.4 - 2.6 M 0.87 to 1.01, 2.6 - 3.1 M 0.85 to 1.09 (1588 x 760 -> 1720 23.1 and
    // 25.1), 3.1 - 3.6 M 0.94 to 1.12 (2139 x 800 -> 1512 32.9 and 36.9).  The line is drawn below the first of them that lose.  Both sets of partial
    // sums are needed at once.
    const GemmPlan &p = m.gemm_fwd[0];
    if (short_shrink && product_in_two_launches(p, d->T, d->d_out)) {
        const int n = short_shares(m.hdr, m.slices16, d->d_in, m.short_cap()).n;
        const size_t parts = align_up((size_t)n * m.slices_all * 16 * m.hdr.max_r16 * 4, 256);
        const size_t end = align_up(m.ws.part + parts + (size_t)p.n_split * d->T * d->d_out * 4, 256) + 256;
        if (!fits_scratch || end <= (size_t)PLORA_NOALLOC_SCRATCH_BYTES) {
            m.fwd_parts = parts;
            total[0] = std::max(total[0], end);
        }
    }
    // dX beside the weight gradients: in small tiles alone.  Its partial tiles lie behind theirs, or, where theirs are none, in the
    // place of the skinny ones as otherwise.
    for (int i = 0; i < 2; ++i) {
        const GemmPlan &q = m.gemm_dx[i];
        if (!bf || m.hdr.n_blocks == 0 || q.bm == 0 || q.big_tiles != 0) continue;
        const size_t a_bytes = m.split_dA > 1 ? (size_t)m.split_dA * m.r16_total * d->d_in * 4 : 0;
        const size_t b_bytes = m.split_dB > 1 ? (size_t)m.split_dB * m.r16_total * d->d_out * 4 : 0;
        const size_t at = a_bytes + b_bytes > 0 ? m.ws.wpart + align_up(std::max(a_bytes, b_bytes), 256) : m.ws.gpart;
        const size_t end = align_up(at + split_bytes(q, d->d_in), 256) + 256;
        if (fits_scratch && end > (size_t)PLORA_NOALLOC_SCRATCH_BYTES) continue;
        m.dx_part[i] = at;
        total[i] = std::max(total[i], end);
    }
    // (backward_impl runs a recomputed shrink beside dH where the workspace reaches that far: with an expanded weight where the dense one does)
    const size_t pair_end = m.ws.wpart + (size_t)m.split_dh * m.hdr.n_blocks * kSkinnyRows * m.hdr.max_r16 * 4 + 256;
    if (bf && pair_end <= total[0]) total[1] = std::max(total[1], align_up(pair_end, 256));
    m.ws_nf4 = m.ws;
    m.ws.total = total[0];
    m.ws_nf4.total = total[1];
}

// ---- metadata cache: the last few descriptions and what was derived from them ---------------------
struct CacheEntry {
    std::vector<int64_t> key;
    std::shared_ptr<const HostMeta> meta;
    uint64_t stamp = 0;
};
constexpr int kCacheEntries = 16;
static std::mutex g_cache_mu;
static CacheEntry g_cache[kCacheEntries];
static uint64_t g_cache_clock = 0;

static void key_of(const plora_desc *d, std::vector<int64_t> &k)
{
    k.clear();
    k.reserve(6 + 2 * (size_t)d->n_seg + (size_t)d->n_adapters);
    k.push_back(d->T); k.push_back(d->d_in); k.push_back(d->d_out); k.push_back(d->dtype + 16 * (int64_t)d->w_layout);
    k.push_back(d->n_seg); k.push_back(d->n_adapters);
    for (int32_t s = 0; s < d->n_seg; ++s) { k.push_back(d->seg_off[s + 1]); k.push_back(d->seg_adapter[s]); }
    for (int32_t a = 0; a < d->n_adapters; ++a) k.push_back(d->rank[a]);
}

// The derived metadata of a valid description (from the cache when the same layout was seen lately).
static std::shared_ptr<const HostMeta> meta_of(const plora_desc *d)
{
    thread_local std::vector<int64_t> key;
    key_of(d, key);
    {
        std::lock_guard<std::mutex> lock(g_cache_mu);
        for (CacheEntry &e : g_cache)
            if (e.meta && e.key == key) { e.stamp = ++g_cache_clock; return e.meta; }
    }
    auto fresh = std::make_shared<HostMeta>();
    build_meta(d, *fresh);
    std::lock_guard<std::mutex> lock(g_cache_mu);
    CacheEntry *victim = &g_cache[0];
    for (CacheEntry &e : g_cache)
        if (e.stamp < victim->stamp) victim = &e;
    victim->key = key; victim->meta = fresh; victim->stamp = ++g_cache_clock;
    return fresh;
}

// ---- bench-only kernel timing (declared in plora_bench.h) -------------------------------------------
// Every kernel class of a call is bracketed by a pair of HIP events recorded on the call's own
// stream; pairs come from a pool that is filled while timing is enabled and summed on request.
constexpr int kClasses = 10;
constexpr int kMaxPairs = 16384;
static int g_timing = 0;
static std::vector<hipEvent_t> g_pool;            // 2 events per pair, created on demand
static std::vector<int> g_pair_class;             // class of each recorded pair

struct Bracket {
    int pair; hipStream_t st;
    Bracket(int cls, hipStream_t s) : pair(-1), st(s)
    {
        if (!g_timing || (int)g_pair_class.size() >= kMaxPairs) return;
        pair = (int)g_pair_class.size();
        if ((int)g_pool.size() < 2 * (pair + 1)) {
            hipEvent_t a, b;
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { pair = -1; return; }
            g_pool.push_back(a); g_pool.push_back(b);
        }
        g_pair_class.push_back(cls);
        (void)hipEventRecord(g_pool[2 * pair], st);
    }
    ~Bracket() { if (pair >= 0) (void)hipEventRecord(g_pool[2 * pair + 1], st); }
};

#define PL_TRY(expr) do { hipError_t e__ = (expr); if (e__ != hipSuccess) return PLORA_ERR_HIP; } while (0)

static bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Outputs in memory that the call reads.  Launches that hold several products write some outputs while others still read their
// operands; a caller may have put an output where, one product after the other, nothing reads any more (plora.h says which), and
// such a call runs them one after the other.
struct Span { const void *p; size_t bytes; };
static bool meet(const Span &a, const Span &b)
{
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.p), b0 = reinterpret_cast<uintptr_t>(b.p);
    return a.p && b.p && a.bytes > 0 && b.bytes > 0 && a0 < b0 + b.bytes && b0 < a0 + a.bytes;
}
// grads: dA (width d_in) or dB (width d_out)
static bool meet_any(const plora_desc *d, float *const *grads, int64_t width, const Span &s)
{
    for (int32_t k = 0; k < d->n_adapters; ++k)
        if (meet(Span{grads[k], (size_t)(d->rank[k] * width) * 4}, s)) return true;
    return false;
}

// One call's host state: the cached metadata and the compact description with this call's pointers.
struct Call {
    std::shared_ptr<const HostMeta> m;
    const WorkspaceLayout *L = nullptr;      // the workspace layout of this kind of call (inside *m)
    uint32_t small[kChunkWords];
    std::vector<uint32_t> large;
    const uint32_t *words = nullptr;
};

// Which calls: with a dense W, with one that the call expands, or the stand-alone low-rank ones (no W).
enum class Form { kDense, kNf4, kLoraOnly };

// Checks shared by forward and backward.
static plora_status prepare(const plora_desc *d, const void *x, const void *W, const void *const *A,
                            const void *const *B, float *const *dA, float *const *dB, void *workspace, size_t ws_bytes,
                            Form form, Call &c)
{
    plora_status st = validate(d);
    if (st != PLORA_OK) return st;
    if (!x && d->T > 0) return PLORA_ERR_NULL;
    if (!W && form != Form::kLoraOnly) return PLORA_ERR_NULL;
    if (d->n_adapters > 0 && (!A || !B)) return PLORA_ERR_NULL;
    for (int32_t k = 0; k < d->n_adapters; ++k) {
        if (!A[k] || !B[k]) return PLORA_ERR_NULL;
        if (misaligned(A[k]) || misaligned(B[k])) return PLORA_ERR_ALIGN;
    }
    if (misaligned(x) || misaligned(W)) return PLORA_ERR_ALIGN;
    c.m = meta_of(d);
    c.L = form == Form::kLoraOnly ? &c.m->ws_lora : form == Form::kNf4 ? &c.m->ws_nf4 : &c.m->ws;
    if (!workspace || ws_bytes < c.L->total) return PLORA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return PLORA_ERR_ALIGN;
    uint32_t *w = c.small;
    if (c.m->n_words > kChunkWords) { c.large.resize((size_t)c.m->n_words); w = c.large.data(); }
    fill_desc_words(d, c.m->hdr.n_blocks, A, B, dA, dB, static_cast<const char *>(workspace) + c.L->at, c.m->order_is_identity, w);
    c.words = w;
    return PLORA_OK;
}

static MetaView device_view(const HostMeta &m, const WorkspaceLayout &L, char *ws)
{
    return view_of(tables_at(ws + L.meta, m.layout));
}

// Base GEMM of one direction.  w_rows_contract: the contraction index is W's row index.
static hipError_t run_gemm(const HostMeta &m, const WorkspaceLayout &L, char *ws, const GemmPlan &plan, bool w_rows_contract, int64_t Kd,
                           int64_t N, const void *S, const void *W, void *C, bool accumulate, hipStream_t st)
{
    const MetaView mv = device_view(m, L, ws);
    if (plan.big_tiles > 0) {
        const hipError_t e = launch_gemm_bf16(mv, m.hdr, w_rows_contract, Kd, N, S, W, ws + L.hb, ws + L.ap, ws + L.zero, C, accumulate,
                                              plan.big_tiles, reinterpret_cast<float *>(ws + L.gpart), plan.bm == 0 ? plan.n_split : 1, st);
        if (e != hipSuccess || plan.bm == 0) return e;
    }
    return launch_gemm_small_bf16(plan, mv, m.hdr, w_rows_contract, Kd, N, S, W, ws + L.hb, ws + L.ap, ws + L.zero, C, accumulate,
                                  reinterpret_cast<float *>(ws + L.gpart), st);
}

// Whether the low-rank products of an fp32 call fit the preparation launch (workgroups in 31 bits, two products).
static bool f32_units_fit(const HostMeta &m) { return (int64_t)m.hdr.n_blocks * kShortSlices * (m.hdr.max_r16 / 16) <= (1 << 22); }

// Steps of a call, so that a grouped call can run a fused pass of its own between them (a plain call runs them all).
enum : unsigned {
    kStepPrep = 1u, kStepShrink = 2u, kStepMain = 4u,      // forward: prep, shrink, GEMM (or stand-alone update)
    kStepDh = 8u, kStepDb = 16u, kStepDa = 32u, kStepDx = 64u,   // backward: prep, shrink, dH, dB, dA, dX
    kStepsAll = 127u
};

// Preparation jobs of a grouped call, launched together once every projection has added its own.
struct PrepList {
    PrepJob job[kMaxGroup];
    std::vector<uint32_t> words[kMaxGroup];
    int n = 0;
    void add(const PrepJob &j)
    {
        words[n].assign(j.desc_host, j.desc_host + j.n_words);       // the description lives in the projection's call frame
        job[n] = j;
        job[n].brief = nullptr; job[n].n_brief = 0;
        job[n].f32 = nullptr; job[n].n_f32 = 0;
        job[n].dh = nullptr;
        job[n].desc_host = words[n].data();
        ++n;
    }
};

// The same of shrink and dH.
struct SkinnyList {
    SkinnyOperands op[kMaxGroup];
    int n = 0;
};

// Weight-gradient products, launched together: of one call, or of every projection of a grouped call.
struct TokcList {
    TokcOperands op[kTokMaxPasses];
    int n = 0;
};
static hipError_t launch_grads(TokcList &l, bool one_by_one, int n_adapters, const void *zero, const GradsDx *dx, hipStream_t st)
{
    const int n = l.n, step = one_by_one ? 1 : n;
    l.n = 0;
    for (int i = 0; i < n; i += step) {
        const hipError_t e = launch_tokcontract_bf16(l.op + i, step, n_adapters, zero, dx, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Forwards in two launches, launched together.
struct ForwardList {
    ShortForward op[kMaxGroup];
    std::vector<uint32_t> words[kMaxGroup];
    int n = 0;
    void add(const ShortForward &f)
    {
        words[n].assign(f.desc_host, f.desc_host + f.n_words);       // the description lives in the projection's call frame
        op[n] = f;
        op[n].desc_host = words[n].data();
        ++n;
    }
};

static plora_status forward_impl(const plora_desc *desc, const void *x, const void *W, const void *const *A,
                                 const void *const *B, void *y, float *h_saved, void *workspace, size_t ws_bytes,
                                 void *hip_stream, Form form = Form::kDense, bool check_only = false, unsigned steps = kStepsAll,
                                 PrepList *later = nullptr, const Nf4Job *nf4 = nullptr, SkinnyList *later_s = nullptr, ForwardList *later_f = nullptr)
{
    const bool lora_only = form == Form::kLoraOnly;
    Call c;
    plora_status ps = prepare(desc, x, W, A, B, nullptr, nullptr, workspace, ws_bytes, form, c);
    if (ps != PLORA_OK) return ps;
    const HostMeta &m = *c.m;
    const WorkspaceLayout &L = *c.L;
    if (!y && desc->T > 0) return PLORA_ERR_NULL;
    if (misaligned(y) || misaligned(h_saved)) return PLORA_ERR_ALIGN;
    if (desc->T == 0 || check_only) return PLORA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);

    const MetaView mv = device_view(m, L, ws);
    const bool lora = m.hdr.n_blocks > 0;
    const bool bf = desc->dtype == PLORA_BF16;
    const bool w_out_in = m.hdr.w_out_in != 0;
    // a short batch: the shrink runs in the preparation launch (not in an NF4 call: its registers would cost the waves that
    // stream the weight, 47 -> 57 us for the two together, and in a launch of its own it is no faster than k_skinny)
    const bool is_short = bf && lora && !nf4 && skinny_is_short(m.hdr, m.slices16, m.r16_total, desc->d_in);
    const bool brief = is_short && !later && (steps & kStepPrep) && (steps & kStepShrink) && m.n_words <= kChunkWords;
    if (brief && !lora_only && m.fwd_parts > 0) {
        float *h_part = reinterpret_cast<float *>(ws + L.part), *y_part = reinterpret_cast<float *>(ws + L.part + m.fwd_parts);
        const ShortForward f{c.words, m.n_words, m.hdr, ws + L.meta, ws + L.zero, x, W, y, h_saved, h_part, y_part, m.slices_all,
                             short_shares(m.hdr, m.slices16, desc->d_in, m.short_cap()), m.gemm_fwd[0]};
        if (later_f) { later_f->add(f); return PLORA_OK; }
        Bracket b(0, st);
        PL_TRY(launch_short_forward(&f, 1, st));
        return PLORA_OK;
    }
    const SkinnyOperands shrink{mv, m.hdr, 0, x, desc->d_in, ws + L.at, reinterpret_cast<float *>(ws + L.part), is_short ? m.short_cap() : m.split_shrink,
                                reinterpret_cast<unsigned long long *>(ws + L.flags), m.slices16, h_saved, ws + L.hb, nullptr, false, is_short, lora_only,
                                m.mean_r16};
    // the fp32 path: its shrink runs in the preparation launch as well
    float *hf = h_saved ? h_saved : reinterpret_cast<float *>(ws + L.hf);
    const bool f32_early = !bf && lora && !later && !nf4 && (steps & kStepPrep) && (steps & kStepShrink) && m.n_words <= kChunkWords && f32_units_fit(m);
    const F32LowRank f32_h{static_cast<const float *>(x), hf, desc->d_in, 0};
    if (steps & kStepPrep) {
        const PrepJob job{c.words, m.n_words, m.max_rank, m.hdr, ws + L.meta, reinterpret_cast<uint32_t *>(ws + L.desc), ws + L.zero,
                          ws + L.at, ws + L.ap, bf && lora && !brief, false, bf && lora && (w_out_in || lora_only), nullptr, nullptr,
                          &shrink, brief ? 1 : 0, &f32_h, f32_early ? 1 : 0, nullptr};
        if (later) later->add(job);
        else if (nf4) { Bracket b(9, st); PL_TRY(launch_prep_nf4(job, *nf4, desc->dtype == PLORA_BF16, st)); }
        else { Bracket b(6, st); PL_TRY(launch_prep(&job, 1, st)); }
    }

    if (desc->dtype == PLORA_F32) {
        const float *xf = static_cast<const float *>(x);
        if (lora && !f32_early && (steps & kStepShrink)) { Bracket b(2, st); PL_TRY(launch_f32_lowrank(mv, m.hdr, 0, xf, desc->d_in, hf, st)); }
        if (!(steps & kStepMain)) return PLORA_OK;
        if (lora_only) {
            Bracket b(8, st);
            PL_TRY(launch_f32_expand(mv, m.hdr, true, static_cast<float *>(y), hf, st));
            return PLORA_OK;
        }
        { Bracket b(0, st);
          PL_TRY(launch_f32_gemm(mv, m.hdr, true, xf, static_cast<const float *>(W), hf, static_cast<float *>(y), false, st)); }
        return PLORA_OK;
    }

    void *hb = ws + L.hb;
    if (lora && !brief && (steps & kStepShrink)) {
        if (later_s) later_s->op[later_s->n++] = shrink;
        else { Bracket b(2, st); PL_TRY(launch_skinny_bf16(&shrink, 1, ws + L.zero, st)); }
    }
    if (!(steps & kStepMain)) return PLORA_OK;
    if (lora_only) {
        // the padded buffer holds B_k^T [d_out][rp]
        Bracket b(8, st);
        PL_TRY(launch_expand_bf16(mv, m.hdr, y, desc->d_out, hb, ws + L.ap, ws + L.zero, st));
        return PLORA_OK;
    }
    { Bracket b(0, st);
      PL_TRY(run_gemm(m, L, ws, m.gemm_fwd[nf4 != nullptr], !w_out_in, desc->d_in, desc->d_out, x, W, y, false, st)); }
    return PLORA_OK;
}

static plora_status backward_impl(const plora_desc *desc, const void *x, const void *W, const void *const *A,
                                  const void *const *B, const void *dy, const float *h_saved, void *dx, float *const *dA,
                                  float *const *dB, void *workspace, size_t ws_bytes, void *hip_stream, Form form = Form::kDense,
                                  bool check_only = false, unsigned steps = kStepsAll, bool dx_accumulate = false,
                                  PrepList *later = nullptr, const Nf4Job *nf4 = nullptr, TokcList *later_w = nullptr,
                                  SkinnyList *later_s = nullptr)
{
    const bool lora_only = form == Form::kLoraOnly, want_w = (dA != nullptr) || (dB != nullptr);
    if (desc && want_w && desc->n_adapters > 0 && (!dA || !dB)) {
        plora_status v = validate(desc);
        return v != PLORA_OK ? v : PLORA_ERR_NULL;
    }
    Call c;
    plora_status ps = prepare(desc, x, W, A, B, want_w ? dA : nullptr, want_w ? dB : nullptr, workspace, ws_bytes, form, c);
    if (ps != PLORA_OK) return ps;
    const HostMeta &m = *c.m;
    const WorkspaceLayout &L = *c.L;
    if (!dy && desc->T > 0) return PLORA_ERR_NULL;
    if (misaligned(dy) || misaligned(dx) || misaligned(h_saved)) return PLORA_ERR_ALIGN;
    if (want_w && desc->n_adapters > 0) {
        for (int32_t k = 0; k < desc->n_adapters; ++k) {
            if (!dA[k] || !dB[k]) return PLORA_ERR_NULL;
            if (misaligned(dA[k]) || misaligned(dB[k])) return PLORA_ERR_ALIGN;
        }
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    const bool lora = m.hdr.n_blocks > 0;
    const bool any_w = want_w && desc->n_adapters > 0;
    if ((desc->T == 0 && !any_w) || check_only) return PLORA_OK;

    const MetaView mv = device_view(m, L, ws);
    const bool bf = desc->dtype == PLORA_BF16;
    const bool need_shrink = any_w && !h_saved;
    // a short batch: dH, and the shrink where h was not saved, run in the preparation launch; both at once share the room for
    // partial tiles and flags
    const bool may_short = bf && lora && !nf4;
    const bool short_sh = may_short && skinny_is_short(m.hdr, m.slices16, m.r16_total, desc->d_in), short_dh = may_short && skinny_is_short(m.hdr, m.slices16, m.r16_total, desc->d_out);
    const bool may_brief = !later && (steps & kStepPrep) && m.n_words <= kChunkWords && m.skinny_cap > 1;
    const bool brief_sh = may_brief && short_sh && need_shrink && (steps & kStepShrink), brief_dh = may_brief && short_dh && (steps & kStepDh);
    const bool f32_early = !bf && lora && !later && !nf4 && (steps & kStepsAll) == kStepsAll && m.n_words <= kChunkWords && f32_units_fit(m);
    float *part = reinterpret_cast<float *>(ws + L.part);
    unsigned long long *flags = reinterpret_cast<unsigned long long *>(ws + L.flags);
    const SkinnyOperands shrink{mv, m.hdr, 0, x, desc->d_in, ws + L.at, part, short_sh ? m.short_cap() : m.split_shrink, flags, m.slices16,
                                nullptr, nullptr, ws + L.zt_h, false, short_sh, lora_only, m.mean_r16};
    SkinnyOperands dh{mv, m.hdr, 1, dy, desc->d_out, nullptr, part, short_dh ? m.short_cap() : m.split_dh, flags, m.slices16,
                      nullptr, ws + L.hb, any_w ? ws + L.zt_g : nullptr, true, short_dh, lora_only, m.mean_r16};
    if (brief_sh && brief_dh) {
        dh.part += (size_t)m.short_cap() * m.hdr.n_blocks * kSkinnyRows * m.hdr.max_r16;
        dh.flags += flag_count(m.hdr);
    }
    // both in one launch (and one finishing launch) where neither is short: dH's partial tiles lie where those of the weight
    // gradients come later, so neither product is split less than alone and the sums are the same.  1024 tokens, 4096 and
    // 14336 columns 33.3 -> 21.6 us
    const bool pair = lora && bf && !later && need_shrink && (steps & kStepShrink) && (steps & kStepDh) && !short_sh && !short_dh &&
                      (size_t)m.split_dh * m.hdr.n_blocks * kSkinnyRows * m.hdr.max_r16 * 4 <= L.total - 256 - L.wpart;
    if (pair) dh.part = reinterpret_cast<float *>(ws + L.wpart);
    // dH that is not short shares the launch of the preparation, up to eight workgroups of that for one of dH: they then have its LDS, two
    // or three on a compute unit.  Whole steps, us, apart and together: 8192 tokens, 1024 -> 1024, 16 adapters (256 packing, 213 of dH) 122 and 114;
    // 4096 tokens, 2048 -> 2048, 8 adapters 148 and 142; 16384 tokens, 4096 -> 14336, low-rank calls alone 789 and 783; 8192 tokens, 8192 ->
    // 28672, 32 adapters (6 for one) 6139 and 6131; 4096 tokens, 8192 -> 8192, 32 adapters (10 for one) 1097 and 1105
    const int64_t pack_wgs = dx ? (desc->d_in + 63) / 64 * m.hdr.n_adapters : 0;
    const bool early_dh = lora && bf && !later && !nf4 && (steps & kStepPrep) && (steps & kStepDh) && !short_dh && !pair && !need_shrink &&
                          m.n_words <= kChunkWords && pack_wgs <= 8 * (int64_t)m.hdr.n_blocks * m.split_dh;
    if (steps & kStepPrep) {
        const bool tr = bf && lora && any_w && h_saved;
        SkinnyOperands brief[kPrepShort];
        int n_brief = 0;
        if (brief_sh) brief[n_brief++] = shrink;
        if (brief_dh) brief[n_brief++] = dh;
        F32LowRank f32[kPrepShort];
        int n_f32 = 0;
        if (f32_early && need_shrink) f32[n_f32++] = F32LowRank{static_cast<const float *>(x), reinterpret_cast<float *>(ws + L.hf), desc->d_in, 0};
        if (f32_early) f32[n_f32++] = F32LowRank{static_cast<const float *>(dy), reinterpret_cast<float *>(ws + L.gf), desc->d_out, 1};
        // the low-rank operand of the dX GEMM: padded A_k, or - W stored [d_out][d_in] - the packed A_k^T
        // (the stand-alone low-rank update always reads the padded A_k)
        const bool dx_ap = dx != nullptr && (lora_only || !m.hdr.w_out_in), dx_at = dx != nullptr && !lora_only && m.hdr.w_out_in;
        const PrepJob job{c.words, m.n_words, m.max_rank, m.hdr, ws + L.meta, reinterpret_cast<uint32_t *>(ws + L.desc), ws + L.zero,
                          ws + L.at, ws + L.ap, bf && lora && ((need_shrink && !brief_sh) || dx_at), bf && lora && dx_ap, false,
                          tr ? h_saved : nullptr, tr ? ws + L.zt_h : nullptr, brief, n_brief, f32, n_f32, early_dh ? &dh : nullptr};
        if (later) later->add(job);
        else if (nf4) { Bracket b(9, st); PL_TRY(launch_prep_nf4(job, *nf4, desc->dtype == PLORA_BF16, st)); }
        else { Bracket b(early_dh ? 3 : 6, st); PL_TRY(launch_prep(&job, 1, st)); }
    }

    if (desc->dtype == PLORA_F32) {
        const float *xf = static_cast<const float *>(x), *dyf = static_cast<const float *>(dy);
        float *gf = reinterpret_cast<float *>(ws + L.gf);
        const float *hf = h_saved;
        if (lora && any_w && !hf) {
            float *hw = reinterpret_cast<float *>(ws + L.hf);
            if (!f32_early && (steps & kStepShrink)) { Bracket b(2, st); PL_TRY(launch_f32_lowrank(mv, m.hdr, 0, xf, desc->d_in, hw, st)); }
            hf = hw;
        }
        if (lora && !f32_early && (steps & kStepDh)) { Bracket b(3, st); PL_TRY(launch_f32_lowrank(mv, m.hdr, 1, dyf, desc->d_out, gf, st)); }
        const bool one = any_w && dx && desc->T > 0 && !lora_only && !dx_accumulate && (steps & kStepDb) && (steps & kStepDx) && f32_bwd_fits(m.hdr, m.max_rank);
        const Span dx_span{dx, (size_t)(desc->T * desc->d_in) * 4};
        if (one && !meet(dx_span, Span{x, dx_span.bytes}) && !meet(dx_span, Span{hf, m.h_elems * 4})) {
            Bracket b(1, st);
            PL_TRY(launch_f32_bwd(mv, m.hdr, m.max_rank, xf, gf, dyf, hf, static_cast<const float *>(W), static_cast<float *>(dx), st));
            return PLORA_OK;
        }
        if (any_w) {
            // (an fp32 call always runs the two steps together: grouped calls do not fuse fp32 projections)
            if (steps & kStepDb) { Bracket b(4, st); PL_TRY(launch_f32_wgrad(mv, m.hdr, m.max_rank, xf, gf, dyf, hf, st)); }
        }
        if (!(steps & kStepDx)) return PLORA_OK;
        if (dx && desc->T > 0 && lora_only) {
            Bracket b(8, st);
            PL_TRY(launch_f32_expand(mv, m.hdr, false, static_cast<float *>(dx), gf, st));
        } else if (dx && desc->T > 0) {
            Bracket b(1, st);
            PL_TRY(launch_f32_gemm(mv, m.hdr, false, dyf, static_cast<const float *>(W), gf, static_cast<float *>(dx), dx_accumulate, st));
        }
        return PLORA_OK;
    }

    void *ap = ws + L.ap, *gb = ws + L.hb;
    void *zt_h = ws + L.zt_h, *zt_g = ws + L.zt_g;
    float *wpart = reinterpret_cast<float *>(ws + L.wpart);
    if (pair) {
        const SkinnyOperands both[2] = {shrink, dh};
        Bracket b(3, st);
        PL_TRY(launch_skinny_bf16(both, 2, ws + L.zero, st));
    } else if (lora) {
        if (need_shrink && !brief_sh && (steps & kStepShrink)) {
            if (later_s) later_s->op[later_s->n++] = shrink;
            else { Bracket b(2, st); PL_TRY(launch_skinny_bf16(&shrink, 1, ws + L.zero, st)); }
        }
        if (!brief_dh && !early_dh && (steps & kStepDh)) {
            if (later_s) later_s->op[later_s->n++] = dh;
            else { Bracket b(3, st); PL_TRY(launch_skinny_bf16(&dh, 1, ws + L.zero, st)); }
        }
    }
    if (any_w) {
        // dB and dA in one launch; the smaller set of partial tiles lies where the skinny ones were (summed by now)
        TokcList own;
        TokcList &list = later_w ? *later_w : own;
        if (steps & kStepDb) list.op[list.n++] = TokcOperands{mv, dy, zt_h, desc->d_out, m.small_part_is_dB ? part : wpart, m.split_dB, m.r16_total, m.hdr.max_r16, false, m.hdr.T};
        if (steps & kStepDa) list.op[list.n++] = TokcOperands{mv, x, zt_g, desc->d_in, m.small_part_is_dB ? wpart : part, m.split_dA, m.r16_total, m.hdr.max_r16, true, m.hdr.T};
        if (own.n > 0) {
            const Span x_span{x, (size_t)(desc->T * desc->d_in) * 2};
            const bool one_by_one = meet_any(desc, dA, desc->d_in, Span{dy, (size_t)(desc->T * desc->d_out) * 2});
            const GemmPlan &plan = m.gemm_dx[nf4 != nullptr];
            // dX in the same launch; not where it would be written over the x that dA reads
            const bool joint = m.dx_part[nf4 != nullptr] > 0 && own.n == 2 && !one_by_one && dx && desc->T > 0 && !lora_only && !dx_accumulate &&
                               (steps & kStepDx) && !meet(Span{dx, x_span.bytes}, x_span);
            const GradsDx gd{mv, m.hdr, plan, m.hdr.w_out_in != 0, desc->d_out, desc->d_in, dy, W, gb, ap, ws + L.zero, dx,
                             reinterpret_cast<float *>(ws + m.dx_part[nf4 != nullptr])};
            Bracket b(joint ? 1 : 4, st);
            PL_TRY(launch_grads(own, one_by_one, m.hdr.n_adapters, ws + L.zero, joint ? &gd : nullptr, st));
            if (joint) return PLORA_OK;
        }
    }
    if (!(steps & kStepDx)) return PLORA_OK;
    if (dx && desc->T > 0 && lora_only) {
        // the padded buffer holds A_k [d_in][rp]
        Bracket b(8, st);
        PL_TRY(launch_expand_bf16(mv, m.hdr, dx, desc->d_in, gb, ap, ws + L.zero, st));
    } else if (dx && desc->T > 0) {
        Bracket b(1, st);
        PL_TRY(run_gemm(m, L, ws, m.gemm_dx[nf4 != nullptr], m.hdr.w_out_in != 0, desc->d_out, desc->d_in, dy, W, dx, dx_accumulate, st));
    }
    return PLORA_OK;
}

// ---- grouped calls: several projections on one x -------------------------------------------------------
// Each projection keeps a workspace of its own inside the group's (so every table and side buffer is where the plain
// call would put it); behind them lies the partial-tile region of the fused passes.  Projections are fused in cells:
// consecutive projections whose ranks, each padded to 16, sum to at most PLORA_MAX_RANK for every adapter, and whose
// plain calls split the shrink alike.
struct GroupPlan {
    int n = 0;
    std::shared_ptr<const HostMeta> m[kMaxGroup];
    size_t ws_off[kMaxGroup] = {};
    int cell_of[kMaxGroup] = {};      // cell index of each projection
    int n_cells = 0;
    size_t part_off = 0, part_bytes = 0, total = 0;
};

struct CellShape { int max_r16 = 0, r16_total = 0; };

// Fused ranks of the projections in `members` (indices into the plan).
static CellShape cell_shape(const GroupPlan &gp, const int *members, int n_members)
{
    CellShape c;
    const int n_ad = gp.m[0]->hdr.n_adapters;
    for (int k = 0; k < n_ad; ++k) {
        int sum = 0;
        for (int i = 0; i < n_members; ++i) sum += gp.m[members[i]]->t.ad[k].r16;
        c.max_r16 = std::max(c.max_r16, sum);
        c.r16_total += sum;
    }
    return c;
}

// Partial tiles of the fused passes of one cell: the most that any two or more of its projections need together.  (A call may
// leave projections out of a pass, and fewer rank rows per adapter can mean more splits of the dA pass, so the whole cell is
// not the largest.)
static size_t cell_part_bytes(const GroupPlan &gp, const plora_desc *d0, const int *cell, int n_cell)
{
    size_t most = 0;
    for (unsigned mask = 1; mask < (1u << n_cell); ++mask) {
        int members[kMaxGroup], nm = 0;
        for (int i = 0; i < n_cell; ++i)
            if (mask >> i & 1u) members[nm++] = cell[i];
        if (nm < 2) continue;
        const CellShape c = cell_shape(gp, members, nm);
        MetaHeader hv = gp.m[members[0]]->hdr;
        hv.max_r16 = c.max_r16;
        const size_t shrink = (size_t)gp.m[members[0]]->split_shrink * hv.n_blocks * kSkinnyRows * c.max_r16 * 4;
        const int sp = tokc_splits(hv, d0->d_in, 0, gp.m[0]->n_active);
        const size_t da = sp > 1 ? (size_t)sp * c.r16_total * d0->d_in * 4 : 0;
        most = std::max(most, std::max(shrink, da));
    }
    return most;
}

static plora_status plan_group(const plora_group *g, GroupPlan &gp)
{
    if (!g) return PLORA_ERR_NULL;
    if (g->n_proj < 1 || g->n_proj > PLORA_MAX_GROUP) return PLORA_ERR_GROUP;
    if (!g->desc) return PLORA_ERR_NULL;
    const plora_desc *d0 = &g->desc[0];
    for (int p = 0; p < g->n_proj; ++p) {
        const plora_desc *d = &g->desc[p];
        plora_status st = validate(d);
        if (st != PLORA_OK) return st;
        if (d->dtype != d0->dtype || d->T != d0->T || d->d_in != d0->d_in || d->n_seg != d0->n_seg || d->n_adapters != d0->n_adapters)
            return PLORA_ERR_GROUP;
        for (int32_t s = 0; s < d->n_seg; ++s)
            if (d->seg_off[s + 1] != d0->seg_off[s + 1] || d->seg_adapter[s] != d0->seg_adapter[s]) return PLORA_ERR_GROUP;
    }
    gp.n = g->n_proj;
    size_t o = 0;
    for (int p = 0; p < gp.n; ++p) {
        gp.m[p] = meta_of(&g->desc[p]);
        gp.ws_off[p] = o;
        o = align_up(o + gp.m[p]->ws.total, 256);
    }
    // cells (bf16 with adapters only: the fp32 path is not fused)
    const bool fuse = d0->dtype == PLORA_BF16 && gp.m[0]->hdr.n_blocks > 0;
    int members[kMaxGroup], nm = 0, cell = 0;
    size_t part = 0;
    for (int p = 0; p < gp.n; ++p) {
        members[nm] = p;
        // (a fused shrink sums in the order of the plain calls, so its projections split the contraction alike)
        if (nm > 0 && (!fuse || cell_shape(gp, members, nm + 1).max_r16 > PLORA_MAX_RANK ||
                       gp.m[p]->split_shrink != gp.m[members[0]]->split_shrink)) {
            part = std::max(part, cell_part_bytes(gp, d0, members, nm));
            ++cell; members[0] = p; nm = 0;
        }
        gp.cell_of[p] = cell;
        ++nm;
    }
    part = std::max(part, cell_part_bytes(gp, d0, members, nm));
    gp.n_cells = cell + 1;
    gp.part_off = o;
    gp.part_bytes = part;
    gp.total = align_up(o + part, 256) + 256;
    return PLORA_OK;
}

// A projection whose plain call takes the routine for short batches takes it here too, and is not fused.
static bool short_shrink(const GroupPlan &gp, int p, const plora_desc *d0) { return skinny_is_short(gp.m[p]->hdr, gp.m[p]->slices16, gp.m[p]->r16_total, d0->d_in); }

// The fused view of the projections `members` of the plan (all of one cell); small: which side buffer the pass gathers.
static void group_view(const GroupPlan &gp, char *ws, const int *members, int nm, bool small_is_at, GroupView &gv, MetaHeader &hv)
{
    const CellShape c = cell_shape(gp, members, nm);
    gv.n_proj = nm; gv.max_r16 = c.max_r16; gv.r16_total = c.r16_total; gv.reserved = 0;
    for (int i = 0; i < kMaxGroup; ++i) {
        const int p = members[i < nm ? i : 0];
        const HostMeta &m = *gp.m[p];
        char *w = ws + gp.ws_off[p];
        gv.mv[i] = device_view(m, m.ws, w);
        gv.small[i] = reinterpret_cast<const uint16_t *>(w + (small_is_at ? m.ws.at : m.ws.zt_g));
    }
    hv = gp.m[members[0]]->hdr;
    hv.max_r16 = c.max_r16;
}

static plora_status group_forward(const plora_group *g, const void *x, const void *const *W, const void *const *const *A,
                                  const void *const *const *B, void *const *y, float *const *h_saved, void *workspace,
                                  size_t ws_bytes, void *hip_stream)
{
    GroupPlan gp;
    plora_status ps = plan_group(g, gp);
    if (ps != PLORA_OK) return ps;
    if (!W || !y || (g->desc[0].n_adapters > 0 && (!A || !B))) return PLORA_ERR_NULL;
    if (!workspace || ws_bytes < gp.total) return PLORA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return PLORA_ERR_ALIGN;
    char *ws = static_cast<char *>(workspace);
    PrepList preps;
    SkinnyList shrinks;
    auto run = [&](int p, bool check, unsigned steps) {
        return forward_impl(&g->desc[p], x, W[p], A ? A[p] : nullptr, B ? B[p] : nullptr, y[p], h_saved ? h_saved[p] : nullptr,
                            ws + gp.ws_off[p], gp.m[p]->ws.total, hip_stream, Form::kDense, check, steps, &preps, nullptr, &shrinks);
    };
    for (int p = 0; p < gp.n; ++p)
        if ((ps = run(p, true, kStepsAll)) != PLORA_OK) return ps;
    if (g->desc[0].T == 0) return PLORA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const plora_desc *d0 = &g->desc[0];
    bool fused[kMaxGroup] = {};
    for (int p = 0; p < gp.n; ++p)
        for (int q = 0; q < gp.n; ++q)
            fused[p] = fused[p] || (q != p && gp.cell_of[q] == gp.cell_of[p] && !short_shrink(gp, p, d0) && !short_shrink(gp, q, d0));
    // Projections whose plain call takes two launches in all take those together, and no step of the group's.  Where others need these
    // steps anyway, unsplit products do so only up to 2.5 M sums in all (their bits are the same either way): 43 such groups, us, together
    // and not: 461 x 1024 -> 5408, 1352, 1352 (1.25 M) 184 and 199, 1575 x 1792 -> 2944, 736, 736 (2.3 M) 179 and 186, 3183 x 1144 -> 1664, 416, 416
    // (2.6 M) 173 and 168, 1240 x 864 -> 4904, 1224, 1224 (3.0 M) 230 and 215, 3684 x 640 -> 2304, 576, 576 (4.2 M) 214 and 188.  Groups that take the
    // two launches whole gain up to the largest there are (4.4 M, 1008 x 1536 -> 2176, 2176 133 and 141).
    bool whole[kMaxGroup], all_whole = true;
    int64_t sums = 0;
    for (int p = 0; p < gp.n; ++p) {
        const HostMeta &m = *gp.m[p];
        all_whole = all_whole && m.fwd_parts > 0;
        if (m.fwd_parts > 0 && m.gemm_fwd[0].n_split == 1) sums += d0->T * g->desc[p].d_out;
    }
    ForwardList wholes;
    for (int p = 0; p < gp.n; ++p) {
        whole[p] = gp.m[p]->fwd_parts > 0 && (all_whole || gp.m[p]->gemm_fwd[0].n_split > 1 || sums <= 2500000);
        ps = whole[p] ? forward_impl(&g->desc[p], x, W[p], A ? A[p] : nullptr, B ? B[p] : nullptr, y[p], h_saved ? h_saved[p] : nullptr,
                                     ws + gp.ws_off[p], gp.m[p]->ws.total, hip_stream, Form::kDense, false, kStepsAll, nullptr, nullptr, nullptr, &wholes)
                      : run(p, false, kStepPrep);
        if (ps != PLORA_OK) return ps;
    }
    if (wholes.n > 0) { Bracket b(0, st); PL_TRY(launch_short_forward(wholes.op, wholes.n, st)); }
    if (preps.n > 0) { Bracket b(6, st); PL_TRY(launch_prep(preps.job, preps.n, st)); }
    for (int p = 0; p < gp.n; ++p)
        if (!fused[p] && !whole[p] && (ps = run(p, false, kStepShrink)) != PLORA_OK) return ps;
    if (shrinks.n > 0) { Bracket b(2, st); PL_TRY(launch_skinny_bf16(shrinks.op, shrinks.n, ws + gp.ws_off[0] + gp.m[0]->ws.zero, st)); }
    for (int c = 0; c < gp.n_cells; ++c) {
        int members[kMaxGroup], nm = 0;
        for (int p = 0; p < gp.n; ++p)
            if (gp.cell_of[p] == c && fused[p]) members[nm++] = p;
        if (nm < 2) continue;
        GroupView gv; MetaHeader hv;
        group_view(gp, ws, members, nm, true, gv, hv);
        float *hf[kMaxGroup] = {}; void *hb[kMaxGroup] = {}; void *zt[kMaxGroup] = {};
        for (int i = 0; i < nm; ++i) {
            hf[i] = h_saved ? h_saved[members[i]] : nullptr;
            hb[i] = ws + gp.ws_off[members[i]] + gp.m[members[i]]->ws.hb;
        }
        Bracket b(2, st);
        PL_TRY(launch_skinny_group(gv, hv, x, g->desc[0].d_in, ws + gp.ws_off[members[0]] + gp.m[members[0]]->ws.zero,
                                   reinterpret_cast<float *>(ws + gp.part_off), gp.part_bytes, gp.m[members[0]]->split_shrink, hf, hb, zt, st));
    }
    for (int p = 0; p < gp.n; ++p)
        if (!whole[p] && (ps = run(p, false, kStepMain)) != PLORA_OK) return ps;
    return PLORA_OK;
}

static plora_status group_backward(const plora_group *g, const void *x, const void *const *W, const void *const *const *A,
                                   const void *const *const *B, const void *const *dy, const float *const *h_saved,
                                   void *const *dx, void *dx_sum, float *const *const *dA, float *const *const *dB,
                                   void *workspace, size_t ws_bytes, void *hip_stream)
{
    GroupPlan gp;
    plora_status ps = plan_group(g, gp);
    if (ps != PLORA_OK) return ps;
    if (!W || !dy || (g->desc[0].n_adapters > 0 && (!A || !B))) return PLORA_ERR_NULL;
    if (dx && dx_sum) return PLORA_ERR_GROUP;            // one or the other
    if (!workspace || ws_bytes < gp.total) return PLORA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return PLORA_ERR_ALIGN;
    char *ws = static_cast<char *>(workspace);
    // dx_sum: every projection's dX GEMM targets the one tensor, the first overwriting it, the others adding to it
    PrepList preps;
    TokcList grads;
    SkinnyList skinny;
    auto run = [&](int p, bool check, unsigned steps) {
        return backward_impl(&g->desc[p], x, W[p], A ? A[p] : nullptr, B ? B[p] : nullptr, dy[p], h_saved ? h_saved[p] : nullptr,
                             dx_sum ? dx_sum : (dx ? dx[p] : nullptr), dA ? dA[p] : nullptr, dB ? dB[p] : nullptr, ws + gp.ws_off[p],
                             gp.m[p]->ws.total, hip_stream, Form::kDense, check, steps, dx_sum != nullptr && p > 0, &preps, nullptr, &grads, &skinny);
    };
    for (int p = 0; p < gp.n; ++p)
        if ((ps = run(p, true, kStepsAll)) != PLORA_OK) return ps;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const plora_desc *d0 = &g->desc[0];
    // which projections want weight gradients, and which of those have to recompute x A_k
    bool want_w[kMaxGroup] = {}, shrink[kMaxGroup] = {}, fuse_s[kMaxGroup] = {}, fuse_a[kMaxGroup] = {};
    for (int p = 0; p < gp.n; ++p) {
        want_w[p] = d0->n_adapters > 0 && ((dA && dA[p]) || (dB && dB[p]));
        shrink[p] = want_w[p] && !(h_saved && h_saved[p]);
    }
    for (int p = 0; p < gp.n; ++p)
        for (int q = 0; q < gp.n; ++q) {
            if (q == p || gp.cell_of[q] != gp.cell_of[p]) continue;
            fuse_s[p] = fuse_s[p] || (shrink[p] && shrink[q] && !short_shrink(gp, p, d0) && !short_shrink(gp, q, d0));
            fuse_a[p] = fuse_a[p] || (want_w[p] && want_w[q]);
        }
    for (int p = 0; p < gp.n; ++p)
        if ((ps = run(p, false, kStepPrep)) != PLORA_OK) return ps;
    if (preps.n > 0) { Bracket b(6, st); PL_TRY(launch_prep(preps.job, preps.n, st)); }
    for (int p = 0; p < gp.n; ++p)
        if (!fuse_s[p] && (ps = run(p, false, kStepShrink)) != PLORA_OK) return ps;
    const void *zero = ws + gp.ws_off[0] + gp.m[0]->ws.zero;
    if (skinny.n > 0) { Bracket b(2, st); PL_TRY(launch_skinny_bf16(skinny.op, skinny.n, zero, st)); skinny.n = 0; }
    for (int c = 0; c < gp.n_cells; ++c) {
        int members[kMaxGroup], nm = 0;
        for (int p = 0; p < gp.n; ++p)
            if (gp.cell_of[p] == c && fuse_s[p]) members[nm++] = p;
        if (nm < 2) continue;
        GroupView gv; MetaHeader hv;
        group_view(gp, ws, members, nm, true, gv, hv);
        float *hf[kMaxGroup] = {}; void *hb[kMaxGroup] = {}; void *zt[kMaxGroup] = {};
        for (int i = 0; i < nm; ++i) zt[i] = ws + gp.ws_off[members[i]] + gp.m[members[i]]->ws.zt_h;
        Bracket b(2, st);
        PL_TRY(launch_skinny_group(gv, hv, x, d0->d_in, ws + gp.ws_off[members[0]] + gp.m[members[0]]->ws.zero,
                                   reinterpret_cast<float *>(ws + gp.part_off), gp.part_bytes, gp.m[members[0]]->split_shrink, hf, hb, zt, st));
    }
    // gradients in the memory of a dy of the group: projection by projection, each with its dX
    bool one_by_one = false;
    for (int p = 0; p < gp.n; ++p) {
        const Span dy_span{dy[p], (size_t)(d0->T * g->desc[p].d_out) * (d0->dtype == PLORA_BF16 ? 2 : 4)};
        for (int q = 0; q < gp.n; ++q)
            one_by_one = one_by_one || (want_w[q] && (meet_any(&g->desc[q], dA[q], d0->d_in, dy_span) ||
                                                      meet_any(&g->desc[q], dB[q], g->desc[q].d_out, dy_span)));
    }
    for (int p = 0; p < gp.n; ++p) {
        if ((ps = run(p, false, kStepDh | kStepDb | (fuse_a[p] ? 0u : kStepDa))) != PLORA_OK) return ps;
        if (!one_by_one && p + 1 < gp.n) continue;
        if (skinny.n > 0) { Bracket b(3, st); PL_TRY(launch_skinny_bf16(skinny.op, skinny.n, zero, st)); skinny.n = 0; }
        // dX of the first projection beside the gradients, as in a plain call (the others, which may add to it, come behind)
        const HostMeta &m0 = *gp.m[0];
        char *ws0 = ws + gp.ws_off[0];
        void *dx0 = dx_sum ? dx_sum : (dx ? dx[0] : nullptr);
        const bool joint = grads.n > 0 && !one_by_one && m0.dx_part[0] > 0 && dx0 && d0->T > 0 &&
                           !meet(Span{dx0, (size_t)(d0->T * d0->d_in) * 2}, Span{x, (size_t)(d0->T * d0->d_in) * 2});
        const GradsDx gd{device_view(m0, m0.ws, ws0), m0.hdr, m0.gemm_dx[0], m0.hdr.w_out_in != 0, d0->d_out, d0->d_in, dy[0], W[0], ws0 + m0.ws.hb,
                         ws0 + m0.ws.ap, ws0 + m0.ws.zero, dx0, reinterpret_cast<float *>(ws0 + m0.dx_part[0])};
        if (grads.n > 0) { Bracket b(joint ? 1 : 4, st); PL_TRY(launch_grads(grads, one_by_one, d0->n_adapters, zero, joint ? &gd : nullptr, st)); }
        for (int q = one_by_one ? p : joint ? 1 : 0; q <= p; ++q)
            if ((ps = run(q, false, kStepDx)) != PLORA_OK) return ps;
    }
    for (int c = 0; c < gp.n_cells; ++c) {
        int members[kMaxGroup], nm = 0;
        for (int p = 0; p < gp.n; ++p)
            if (gp.cell_of[p] == c && fuse_a[p]) members[nm++] = p;
        if (nm < 2) continue;
        GroupView gv; MetaHeader hv;
        group_view(gp, ws, members, nm, false, gv, hv);
        Bracket b(5, st);
        PL_TRY(launch_tokc_group_dA(gv, hv, x, d0->d_in, ws + gp.ws_off[members[0]] + gp.m[members[0]]->ws.zero,
                                    reinterpret_cast<float *>(ws + gp.part_off), gp.part_bytes, tokc_splits(hv, d0->d_in, 0, gp.m[0]->n_active),
                                    gp.m[0]->n_active, st));
    }
    return PLORA_OK;
}

// Scratch memory of plora_linear_fwd_noalloc: one array per GPU, resident from the first use of the
// library on that GPU until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels and copies get the device address looked up once per device.
__device__ __align__(256) unsigned char g_noalloc_scratch[PLORA_NOALLOC_SCRATCH_BYTES];

static plora_status noalloc_scratch(void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *ptr[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PLORA_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_noalloc_scratch)) != hipSuccess || !p) return PLORA_ERR_HIP;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return PLORA_OK;
}

}  // namespace plora

using namespace plora;

// No exception leaves the library: host allocation failures and anything else thrown on the way become a status.
#define PL_GUARDED(fallback, ...) \
    try { __VA_ARGS__ } catch (const std::bad_alloc &) { return fallback; } catch (...) { return fallback; }

extern "C" {

const char *plora_status_string(plora_status st)
{
    switch (st) {
    case PLORA_OK: return "ok";
    case PLORA_ERR_NULL: return "a required pointer is NULL";
    case PLORA_ERR_SHAPE: return "bad T / d_in / d_out (bf16 needs multiples of 8; sizes above the supported range)";
    case PLORA_ERR_SEGMENTS: return "segment offsets must start at 0, end at T and not decrease";
    case PLORA_ERR_ADAPTER: return "adapter id out of range or too many adapters";
    case PLORA_ERR_RANK: return "rank outside [1, PLORA_MAX_RANK]";
    case PLORA_ERR_ALIGN: return "device pointer not 16-byte aligned (workspace: 256)";
    case PLORA_ERR_WORKSPACE: return "workspace missing or too small";
    case PLORA_ERR_UNSUPPORTED: return "unsupported dtype";
    case PLORA_ERR_HIP: return "HIP launch failed";
    case PLORA_ERR_INTERNAL: return "host memory allocation failed or internal error";
    case PLORA_ERR_GROUP: return "grouped call: bad number of projections, or they differ in dtype, T, d_in, segments or adapters";
    }
    return "unknown status";
}

plora_status plora_validate(const plora_desc *desc) { return validate(desc); }

size_t plora_h_elems(const plora_desc *desc)
{
    PL_GUARDED(0,
        if (validate(desc) != PLORA_OK) return 0;
        return meta_of(desc)->h_elems;
    )
}

size_t plora_workspace_bytes(const plora_desc *desc)
{
    PL_GUARDED(0,
        if (validate(desc) != PLORA_OK) return 0;
        return meta_of(desc)->ws.total;
    )
}

int64_t plora_build_metadata(const plora_desc *desc, int32_t block_rows, int64_t *h_off_out,
                             int32_t *blocks_out, int64_t blocks_cap)
{
    PL_GUARDED(-1,
        if (validate(desc) != PLORA_OK || block_rows < 1) return -1;
        const std::shared_ptr<const HostMeta> m = meta_of(desc);
        if (h_off_out) {
            for (int32_t s = 0; s < desc->n_seg; ++s) h_off_out[s] = m->t.seg[s].h_off;
            h_off_out[desc->n_seg] = (int64_t)m->h_elems;
        }
        int64_t n = 0;
        for (int32_t s = 0; s < desc->n_seg; ++s) {
            const SegInfo &g = m->t.seg[s];
            for (int32_t r0 = g.row0; r0 < g.row1; r0 += block_rows) {
                if (blocks_out && n < blocks_cap) {
                    blocks_out[4 * n + 0] = r0;
                    blocks_out[4 * n + 1] = (g.row1 - r0 < block_rows) ? g.row1 - r0 : block_rows;
                    blocks_out[4 * n + 2] = s;
                    blocks_out[4 * n + 3] = g.adapter;
                }
                ++n;
            }
        }
        return n;
    )
}

int plora_debug_metadata(const plora_desc *desc, plora_debug_info *info, void *tables_out, size_t cap)
{
    PL_GUARDED(-1,
        if (validate(desc) != PLORA_OK || !info) return -1;
        HostMeta m;                      // built afresh: the export must not depend on what the cache holds
        build_meta(desc, m);
        std::memset(info, 0, sizeof(*info));
        info->n_tiles = m.layout.n_tiles;
        info->n_seg = m.hdr.n_seg; info->n_adapters = m.hdr.n_adapters;
        info->n_blocks = m.hdr.n_blocks; info->max_r16 = m.hdr.max_r16;
        info->seg_stride = (int32_t)sizeof(SegInfo); info->ad_stride = (int32_t)sizeof(AdapterInfo);
        info->tile_stride = (int32_t)sizeof(GemmTile);
        info->off_hdr = m.layout.hdr; info->off_seg = m.layout.seg; info->off_ad = m.layout.ad;
        info->off_tile = m.layout.tile; info->off_blk_seg = m.layout.blk_seg; info->off_seg_list = m.layout.seg_list;
        info->off_tile_order = m.layout.tile_order;
        info->table_bytes = m.layout.bytes;
        info->shrink_splits = m.split_shrink; info->dh_splits = m.split_dh;
        info->da_splits = m.split_dA; info->da_tile_cols = kTokTileColumns;
        info->db_splits = m.split_dB; info->db_tile_cols = kTokTileColumns;
        info->r16_total = m.r16_total; info->n_active = m.n_active;
        info->ws_zero = m.ws.zero; info->ws_meta = m.ws.meta; info->ws_desc = m.ws.desc; info->ws_at = m.ws.at;
        info->ws_ap = m.ws.ap; info->ws_hb = m.ws.hb; info->ws_zt_h = m.ws.zt_h; info->ws_zt_g = m.ws.zt_g;
        info->ws_hf = m.ws.hf; info->ws_gf = m.ws.gf; info->ws_part = m.ws.part; info->ws_wpart = m.ws.wpart;
        info->ws_total = m.ws.total;
        info->h_elems = m.h_elems;
        info->desc_words = m.n_words;
        for (int i = 0; i < 2; ++i) {
            const GemmPlan &p = i == 0 ? m.gemm_fwd[0] : m.gemm_dx[0];
            info->gemm_rows[i] = p.bm; info->gemm_splits[i] = p.n_split; info->gemm_big_tiles[i] = p.big_tiles;
            const int64_t C = i == 0 ? desc->d_in : desc->d_out;
            const bool is_short = desc->dtype == PLORA_BF16 && skinny_is_short(m.hdr, m.slices16, m.r16_total, C);
            info->short_shares[i] = is_short ? short_shares(m.hdr, m.slices16, C, m.short_cap()).n : 0;
        }
        info->ws_flags = m.ws.flags;
        info->flag_bytes = info->short_shares[0] + info->short_shares[1] > 0 ? 2 * flag_count(m.hdr) * sizeof(unsigned long long) : 0;
        if (tables_out) {
            if (cap < m.layout.bytes) return -1;
            std::memcpy(tables_out, m.image.data(), m.layout.bytes);
        }
        return 0;
    )
}

void plora_set_kernel_timing(int enabled)
{
    g_timing = enabled;
    g_pair_class.clear();
}

int plora_kernel_time(int cls, float *total_ms, int *count)
{
    if (cls < 0 || cls >= kClasses || !total_ms || !count) return -1;
    float tot = 0.f; int n = 0;
    for (size_t p = 0; p < g_pair_class.size(); ++p) {
        if (g_pair_class[p] != cls) continue;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, g_pool[2 * p], g_pool[2 * p + 1]) != hipSuccess) return -1;
        tot += ms; ++n;
    }
    *total_ms = tot; *count = n;
    return 0;
}

plora_status plora_linear_fwd(const plora_desc *desc, const void *x, const void *W,
                              const void *const *A, const void *const *B, void *y, float *h_saved,
                              void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return forward_impl(desc, x, W, A, B, y, h_saved, workspace, ws_bytes, hip_stream);
    )
}

plora_status plora_linear_fwd_noalloc(const plora_desc *desc, const void *x, const void *W,
                                      const void *const *A, const void *const *B, void *y, float *h_saved,
                                      void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        const plora_status v = validate(desc);
        if (v != PLORA_OK) return v;
        if (meta_of(desc)->ws.total > (size_t)PLORA_NOALLOC_SCRATCH_BYTES) return PLORA_ERR_WORKSPACE;
        void *scratch = nullptr;
        const plora_status ps = noalloc_scratch(&scratch);
        if (ps != PLORA_OK) return ps;
        return forward_impl(desc, x, W, A, B, y, h_saved, scratch, PLORA_NOALLOC_SCRATCH_BYTES, hip_stream);
    )
}

static plora_status adamw_collect(const plora_desc *d, const plora_adamw_side *s, bool is_A, const plora_adamw_hparams *hp,
                                  std::vector<AdamwTensor> &out)
{
    if (!s || !s->grad || !s->m || !s->v) return PLORA_ERR_NULL;
    if (!s->param && !s->master) return PLORA_ERR_NULL;
    if (!s->master && d->dtype != PLORA_F32) return PLORA_ERR_NULL;
    for (int32_t k = 0; k < d->n_adapters; ++k) {
        AdamwTensor t;
        t.param = s->param ? s->param[k] : nullptr;
        t.master = s->master ? s->master[k] : nullptr;
        t.grad = s->grad[k]; t.m = s->m[k]; t.v = s->v[k];
        if (!t.grad || !t.m || !t.v || (s->param && !t.param) || (s->master && !t.master)) return PLORA_ERR_NULL;
        if (misaligned(t.param) || misaligned(t.master) || misaligned(t.grad) || misaligned(t.m) || misaligned(t.v))
            return PLORA_ERR_ALIGN;
        t.numel = (uint64_t)d->rank[k] * (uint64_t)(is_A ? d->d_in : d->d_out);
        t.lr = hp[k].lr; t.beta1 = hp[k].beta1; t.beta2 = hp[k].beta2; t.eps = hp[k].eps;
        t.weight_decay = hp[k].weight_decay; t.step = hp[k].step; t.grad_scale = hp[k].grad_scale;
        out.push_back(t);
    }
    return PLORA_OK;
}

plora_status plora_adamw_step(const plora_desc *desc, const plora_adamw_side *A, const plora_adamw_side *B,
                              const plora_adamw_hparams *hp, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        const plora_status v = validate(desc);
        if (v != PLORA_OK) return v;
        if (desc->n_adapters == 0) return PLORA_OK;
        if (!hp) return PLORA_ERR_NULL;
        for (int32_t k = 0; k < desc->n_adapters; ++k)
            if (hp[k].step < 1 || !(hp[k].beta1 >= 0.f && hp[k].beta1 < 1.f) || !(hp[k].beta2 >= 0.f && hp[k].beta2 < 1.f) ||
                !std::isfinite(hp[k].grad_scale))
                return PLORA_ERR_SHAPE;
        std::vector<AdamwTensor> jobs;
        jobs.reserve(2 * (size_t)desc->n_adapters);
        plora_status ps = adamw_collect(desc, A, true, hp, jobs);
        if (ps != PLORA_OK) return ps;
        ps = adamw_collect(desc, B, false, hp, jobs);
        if (ps != PLORA_OK) return ps;
        { Bracket b(7, static_cast<hipStream_t>(hip_stream));
          PL_TRY(launch_adamw(jobs.data(), (int)jobs.size(), desc->dtype == PLORA_BF16, static_cast<hipStream_t>(hip_stream))); }
        return PLORA_OK;
    )
}

plora_status plora_linear_bwd(const plora_desc *desc, const void *x, const void *W,
                              const void *const *A, const void *const *B, const void *dy,
                              const float *h_saved, void *dx, float *const *dA, float *const *dB,
                              void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return backward_impl(desc, x, W, A, B, dy, h_saved, dx, dA, dB, workspace, ws_bytes, hip_stream);
    )
}

// Workspace of the NF4 calls: the ordinary workspace, then the expanded weight.
static size_t nf4_weight_offset(const HostMeta &m) { return align_up(m.ws_nf4.total, 256); }
static size_t nf4_weight_bytes(const plora_desc *d) { return (size_t)d->d_in * (size_t)d->d_out * (d->dtype == PLORA_BF16 ? 2 : 4); }

size_t plora_nf4_workspace_bytes(const plora_desc *desc)
{
    PL_GUARDED(0,
        if (validate(desc) != PLORA_OK || (desc->d_in * desc->d_out) % 64 != 0) return 0;
        return nf4_weight_offset(*meta_of(desc)) + nf4_weight_bytes(desc);
    )
}

plora_status plora_nf4_dequantize(const void *W_codes, const float *W_absmax, int64_t n_elems, int32_t dtype, void *out,
                                  void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        if (dtype != PLORA_BF16 && dtype != PLORA_F32) return PLORA_ERR_UNSUPPORTED;
        if (n_elems < 0 || n_elems % 64 != 0) return PLORA_ERR_SHAPE;
        if (n_elems == 0) return PLORA_OK;
        if (!W_codes || !W_absmax || !out) return PLORA_ERR_NULL;
        if (misaligned(W_codes) || misaligned(W_absmax) || misaligned(out)) return PLORA_ERR_ALIGN;
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        Bracket b(9, st);
        PL_TRY(launch_nf4_dequant(W_codes, W_absmax, n_elems, dtype == PLORA_BF16, out, st));
        return PLORA_OK;
    )
}

// Checks of the NF4 calls that come before anything is enqueued; *w_out = where the expanded weight goes.
static plora_status nf4_prepare(const plora_desc *desc, const void *codes, const float *absmax, void *workspace,
                                size_t ws_bytes, void **w_out, size_t *inner_bytes)
{
    const plora_status v = validate(desc);
    if (v != PLORA_OK) return v;
    if ((desc->d_in * desc->d_out) % 64 != 0) return PLORA_ERR_SHAPE;
    if (!codes || !absmax) return PLORA_ERR_NULL;
    if (misaligned(codes) || misaligned(absmax)) return PLORA_ERR_ALIGN;
    const size_t off = nf4_weight_offset(*meta_of(desc));
    if (!workspace || ws_bytes < off + nf4_weight_bytes(desc)) return PLORA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return PLORA_ERR_ALIGN;
    *w_out = static_cast<char *>(workspace) + off;
    *inner_bytes = off;
    return PLORA_OK;
}

plora_status plora_linear_fwd_nf4(const plora_desc *desc, const void *x, const void *W_codes, const float *W_absmax,
                                  const void *const *A, const void *const *B, void *y, float *h_saved, void *workspace,
                                  size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        void *W = nullptr;
        size_t inner = 0;
        plora_status ps = nf4_prepare(desc, W_codes, W_absmax, workspace, ws_bytes, &W, &inner);
        if (ps != PLORA_OK) return ps;
        // every other argument is checked before the weight is expanded, so that an error enqueues nothing
        ps = forward_impl(desc, x, W, A, B, y, h_saved, workspace, inner, hip_stream, Form::kNf4, true);
        if (ps != PLORA_OK) return ps;
        const Nf4Job job{static_cast<const uint32_t *>(W_codes), W_absmax, W, desc->d_in * desc->d_out};
        return forward_impl(desc, x, W, A, B, y, h_saved, workspace, inner, hip_stream, Form::kNf4, false, kStepsAll, nullptr, &job);
    )
}

plora_status plora_linear_bwd_nf4(const plora_desc *desc, const void *x, const void *W_codes, const float *W_absmax,
                                  const void *const *A, const void *const *B, const void *dy, const float *h_saved, void *dx,
                                  float *const *dA, float *const *dB, void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        void *W = nullptr;
        size_t inner = 0;
        plora_status ps = nf4_prepare(desc, W_codes, W_absmax, workspace, ws_bytes, &W, &inner);
        if (ps != PLORA_OK) return ps;
        ps = backward_impl(desc, x, W, A, B, dy, h_saved, dx, dA, dB, workspace, inner, hip_stream, Form::kNf4, true);
        if (ps != PLORA_OK) return ps;
        const Nf4Job job{static_cast<const uint32_t *>(W_codes), W_absmax, W, desc->d_in * desc->d_out};
        return backward_impl(desc, x, W, A, B, dy, h_saved, dx, dA, dB, workspace, inner, hip_stream, Form::kNf4, false, kStepsAll, false, nullptr,
                             dx && desc->T > 0 ? &job : nullptr);
    )
}

size_t plora_lora_workspace_bytes(const plora_desc *desc)
{
    PL_GUARDED(0,
        if (validate(desc) != PLORA_OK) return 0;
        return meta_of(desc)->ws_lora.total;
    )
}

plora_status plora_lora_fwd(const plora_desc *desc, const void *x, const void *const *A, const void *const *B, void *y,
                            float *h_saved, void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return forward_impl(desc, x, nullptr, A, B, y, h_saved, workspace, ws_bytes, hip_stream, Form::kLoraOnly);
    )
}

plora_status plora_lora_bwd(const plora_desc *desc, const void *x, const void *const *A, const void *const *B,
                            const void *dy, const float *h_saved, void *dx, float *const *dA, float *const *dB,
                            void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return backward_impl(desc, x, nullptr, A, B, dy, h_saved, dx, dA, dB, workspace, ws_bytes, hip_stream, Form::kLoraOnly);
    )
}

size_t plora_group_workspace_bytes(const plora_group *group)
{
    PL_GUARDED(0,
        GroupPlan gp;
        if (plan_group(group, gp) != PLORA_OK) return 0;
        return gp.total;
    )
}

plora_status plora_group_fwd(const plora_group *group, const void *x, const void *const *W, const void *const *const *A,
                             const void *const *const *B, void *const *y, float *const *h_saved, void *workspace,
                             size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return group_forward(group, x, W, A, B, y, h_saved, workspace, ws_bytes, hip_stream);
    )
}

plora_status plora_group_bwd(const plora_group *group, const void *x, const void *const *W, const void *const *const *A,
                             const void *const *const *B, const void *const *dy, const float *const *h_saved,
                             void *const *dx, void *dx_sum, float *const *const *dA, float *const *const *dB,
                             void *workspace, size_t ws_bytes, void *hip_stream)
{
    PL_GUARDED(PLORA_ERR_INTERNAL,
        return group_backward(group, x, W, A, B, dy, h_saved, dx, dx_sum, dA, dB, workspace, ws_bytes, hip_stream);
    )
}

}  // extern "C"
