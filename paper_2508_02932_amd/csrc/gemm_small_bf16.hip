// Base GEMM of the packed multi-LoRA layer for products that have too few 256 x 256 output tiles to
// fill the chip (see gemm_bf16.hip for the large ones; same product, same operands, same low-rank
// extension steps).  Short batches are bound by the stream of W (64 tokens against a 4096 x 4096 weight:
// 34 MB, against 2 GFLOP) or by idle compute units, so the tiles are small and the contraction is
// split over workgroups until about two of them sit on every compute unit.  Against the 256 x 256 kernel:
// 48 tokens, 4096 -> 4096, 83 -> 12 us; 512 tokens, contraction 14336 -> 4096 columns, 250 -> 71 us; 1024 tokens, the
// same, 261 -> 127 us.  What bounds it when the chip is full and W lies in the last-level cache is the traffic from L2 into LDS
// (64 KB per compute unit and stage of 64, 0.95 us: 17 TB/s); with W from HBM, as in a model that walks its layers, it is the
// round trip of a direct load with the few stages that fit beside a second workgroup (512 tokens, 4096 -> 14336, three W slots:
// 65 us from the cache, 72 from HBM).  A loop that reads the operands of the next step during the multiplications, rings of
// 4 and 6 stages and 256 x 128 tiles of eight waves were all no faster, and stages of 32 (64-byte pieces of rows) 20 % slower.
#include "gemm_small.h"

#include <algorithm>

namespace plora {

template <bool FWD, int BM, bool DEEP, bool ACC>
__global__ void __launch_bounds__(256, 2) k_gemm_small(MetaView mv, GemmSmallArgs ga)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    gemm_small_tile<FWD, BM, DEEP, ACC, true>(mv, ga, blockIdx.x, lds);
}

template <bool ACC>
__global__ void __launch_bounds__(256) k_gemm_finish(const float *__restrict__ part, uint16_t *__restrict__ Cout, int64_t n_vec, int n_split)
{
    gemm_finish<ACC>(part, Cout, n_vec, n_split, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

hipError_t launch_gemm_finish(const float *part, void *C, int64_t n, int n_split, bool accumulate, hipStream_t st)
{
    const int64_t n_vec = n / 4;
    const dim3 grid((unsigned)((n_vec + 255) / 256));
    if (accumulate) hipLaunchKernelGGL(k_gemm_finish<true>, grid, dim3(256), 0, st, part, static_cast<uint16_t *>(C), n_vec, n_split);
    else hipLaunchKernelGGL(k_gemm_finish<false>, grid, dim3(256), 0, st, part, static_cast<uint16_t *>(C), n_vec, n_split);
    return hipGetLastError();
}

template <bool FWD, int BM, bool DEEP, bool ACC>
static hipError_t launch_small(const MetaView &mv, const MetaHeader &h, int64_t Kd, int64_t N, const void *S, const void *W,
                               const void *side, const void *ap, const void *zero, void *C, float *part, int n_split, int row_tile0,
                               int slot, hipStream_t st)
{
    constexpr size_t lds = (size_t)(gs_ring_x(BM) * BM + gs_ring_w(BM, DEEP) * GS_BN) * GS_BK * 2;
    const int all256 = (int)((h.T + kGemmTileRows - 1) / kGemmTileRows);
    const int tiles_m = row_tile0 > 0 ? (all256 - row_tile0) * (kGemmTileRows / BM) : (int)((h.T + BM - 1) / BM), tiles_n = (int)((N + GS_BN - 1) / GS_BN);
    auto kern = k_gemm_small<FWD, BM, DEEP, ACC>;
    hipError_t e = allow_full_lds(reinterpret_cast<const void *>(kern), slot);
    if (e != hipSuccess) return e;
    const GemmSmallArgs ga{static_cast<const uint16_t *>(S), static_cast<const uint16_t *>(W), static_cast<const uint16_t *>(side),
                           static_cast<const uint16_t *>(ap), static_cast<const uint16_t *>(zero), static_cast<uint16_t *>(C),
                           n_split > 1 ? part : nullptr, tiles_m, tiles_n, n_split, row_tile0, (int)h.T, (int)Kd, (int)N, (int)h.n_seg};
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n * n_split)), dim3(256), lds, st, mv, ga);
    e = hipGetLastError();
    return e != hipSuccess || n_split <= 1 ? e : launch_gemm_finish(part, C, h.T * N, n_split, ACC, st);
}

template <bool FWD, bool ACC>
static hipError_t dispatch_small(const GemmPlan &p, const MetaView &mv, const MetaHeader &h, int64_t Kd, int64_t N, const void *S,
                                 const void *W, const void *side, const void *ap, const void *zero, void *C, float *part, hipStream_t st)
{
    constexpr int slot = 16 + (FWD ? 1 : 0) + (ACC ? 2 : 0);
    // A third W slot pays where W comes from HBM and four row tiles share it, and costs the better order of the requests: two
    // and three slots, us, W from HBM (in the last-level cache): 4096 -> 14336, 384 tokens 71 and 73 (56 and 64), 512 tokens 80
    // and 72 (60 and 65); 14336 -> 4096, 384 tokens 64 and 66, 512 tokens 85 and 77, 513 to 896 tokens 5 to 9 % slower with
    // three, 1024 tokens 144 and 132 (114 and 123); 8192 -> 8192, 513 to 896 tokens the same to 2 % slower (10 to 20 % slower), 1024
    // tokens 134 and 133 (117 and 127).  The line is drawn for W from HBM, at four row tiles; at eight the split weight gains
    // as well, but the others lose more with W in the cache.
    const bool deep = gemm_small_deep(h.T);
#define PL_GS(BM_, DEEP_, SLOT_) launch_small<FWD, BM_, DEEP_, ACC>(mv, h, Kd, N, S, W, side, ap, zero, C, part, p.n_split, p.big_tiles, slot + 4 * SLOT_, st)
    if (p.bm == 64) return PL_GS(64, false, 0);
    return deep ? PL_GS(128, true, 1) : PL_GS(128, false, 2);
#undef PL_GS
}

hipError_t launch_gemm_small_bf16(const GemmPlan &p, const MetaView &mv, const MetaHeader &h, bool w_rows_contract, int64_t Kd, int64_t N,
                                  const void *S, const void *W, const void *side, const void *ap, const void *zero, void *C,
                                  bool accumulate, float *part, hipStream_t st)
{
    if (w_rows_contract)
        return accumulate ? dispatch_small<true, true>(p, mv, h, Kd, N, S, W, side, ap, zero, C, part, st)
                          : dispatch_small<true, false>(p, mv, h, Kd, N, S, W, side, ap, zero, C, part, st);
    return accumulate ? dispatch_small<false, true>(p, mv, h, Kd, N, S, W, side, ap, zero, C, part, st)
                      : dispatch_small<false, false>(p, mv, h, Kd, N, S, W, side, ap, zero, C, part, st);
}

// Which kernel and split, by the estimated time.  What a stage of 64 contraction elements takes was measured as a
// function of how full the chip is (f = share of the workgroup slots that a round fills; microseconds, d = 4096 and
// 14336, 48 to 16384 tokens, both weight orders):
//   256 x 256 tiles, one workgroup per compute unit     0.92 + 0.78 f     (1.12 at 64 tiles, 1.30 at 128, 1.70 at 256)
//   128 x 128 tiles, two per compute unit               0.38 + 0.62 f     (0.69 at 256 workgroups, 1.00 at 512)
//    64 x 128 tiles, two per compute unit               0.38 + 0.24 f     (0.50 at 256 workgroups, 0.62 at 512)
// (with W in the last-level cache; from HBM the 128 x 128 tiles take up to a third longer, 512 x 4096 -> 14336 80 us against 60
// with two W slots, 72 with the three it runs).
// A split adds the summing launch (4 us) and a write and a read of the fp32 partial tiles.  At the sizes where the
// choice changes both sides were timed (256-tile kernel against the small tiles): 2048 x 4096 -> 4096 83 against 65 us,
// 3072 x 4096 -> 4096 92 against 112 us, 1024 x 4096 -> 14336 103 against 118 us, 512 x 4096 -> 14336 85 against 62 us.
// From three rounds on the small tiles lose (L2 traffic and power: 8192 x 4096 -> 4096 301 against 214 us), so they are
// not considered there.  Between one and eight rounds of the 256-tile kernel a last round that is mostly empty goes to the
// small tiles instead (two launches; us, 256-tile kernel alone and now: 4400 x 4096 -> 4096 184 and 151, 5000 tokens 182 and
// 157, 10000 x 2048 -> 2048 99 and 87, 9000 x 4096 -> 4096 286 and 261, 13000 393 and 366, 6144 183 and 179).  A split keeps four stages or more; the partial tiles stay below 64 MB.
// The 256 x 256 tiles split as well, where that fills three quarters of the compute units: a stage then moves half the bytes into
// LDS for each product.  Estimated as above (0.92 + 0.68 f a stage, the partial tiles at 7.5 TB/s).  Whole backward calls without weight
// gradients, us, T x contraction -> columns, small tiles and split 256-tiles, W from HBM as in a model that walks its layers; r = ratio of the estimates:
//   r 0.80  768 x 28672 -> 4096  236 and 187      0.87  400 x 8296 -> 10368  183 and 112      0.91  768 x 8064 -> 6800   132 and 107
//     0.96  1024 x 14336 -> 4096 163 and 140      0.98  192 x 14336 -> 8192  98 and 91        1.00  512 x 8192 -> 14336  149 and 134
//     1.03  320 x 8192 -> 8192   89 and 83        1.09  330 x 7680 -> 5312   60 and 60        1.11  256 x 4096 -> 8192   51 and 50
//     1.12  320 x 8192 -> 14336  139 and 123      1.16  128 x 4096 -> 8192   39 and 41        1.19  512 x 4096 -> 14336  85 and 87
//     1.22  256 x 4096 -> 14336  68 and 69        1.24  128 x 4096 -> 14336  49 and 61        1.27  320 x 4096 -> 14336  79 and 75
// The line is drawn at 1.12; for a weight that the call itself has just written (w_cached: NF4) at 0.93, for small tiles gain more from the
// last-level cache (forward calls with W there: 1024 x 14336 -> 4096 131 and 133, 512 x 4096 -> 8192 56 and 60).
// Six parts at most: seven and eight at 62 products that six put on three quarters of the compute units or more took 0.95 to 1.24 times as
// long, 1.03 on average (192 x 8192 -> 8192 62 and 71, 400 x 14336 -> 4096 90 and 86).  Below three quarters the best of six and eight parts ran 36
// products in 0.79 to 1.22 times the time of small tiles, 0.97 on average, and the estimate does not tell them apart (128 x 13824 -> 5120, 160
// workgroups, 75 and 63; 192 x 8192 -> 4096, 128 workgroups, 39 and 48).  More than four parts only for weights of 64 MB and more, and below 80 MB
// no column tile that is partly empty: these would gain too (1000 x 14336 -> 2048 99 and 87, 700 x 8200 -> 4104 92 and 78), but what such
// products run on is pinned by tests of the small tiles as it was.
// Not up to 64 tokens, which fill a quarter of a 256-row tile (forward calls: 8 x 8192 -> 8192 32 and 49, 48 x 14336 -> 8192 54 and 77, 26 x
// 6800 -> 8064, seven adapters, 46 and 66).  The first part has all extension steps and walks the segment table for them: from the seventh on
// each costs 2.5 us (1 where the contraction lies along W's rows) more than the small tiles pay, which share them (80 x 8192 -> 8192, one adapter
// 54 and 57, eight of rank 64 57 and 91, sixteen of rank 32 56 and 103; 512 x 8192 -> 14336, 128 adapters, 247 and 344).  With eight row tiles and
// more few segments meet in one of them, and both sides pay alike (3000 x 16384 -> 1024, 128 adapters 267 and 249, 256 adapters 413 and 408; 2000 x
// 8192 -> 2048 128 and 106 for one adapter, 251 and 286 for 256).  And where small tiles in three parts or more would run in two launches
// with the shrink, the launch that the 256-tiles give up is worth 12 us (640 x 8192 -> 4096 69 and 79, 640 x 14336 -> 4096 104 and 112, 330 x 7168 ->
// 7168 67 and 78), unless rows of W share lines of 128 bytes, for which small tiles are slower (72 x 11464 -> 16824 165 and 121, 256 x 6800
// -> 8064 77 and 66).  Of 730 products that the estimates alone would split these lines leave 27 slower than in small tiles, by 2 to 17 % (80 x
// 5120 -> 13824, four adapters, 56 and 65), and keep 8 in small tiles that would gain, up to 11 %; without them 123 were slower, up to 1.83 times.
GemmPlan gemm_plan(const GemmShape &s, double big_split_bytes)
{
    const int64_t T = s.T, Kd = s.Kd, N = s.N;
    constexpr double kCus = 256.0;                             // compute units of an MI355X
    const double nk = (double)((Kd + GS_BK - 1) / GS_BK);
    auto tiles_of = [&](int64_t bm, int64_t bn) { return (double)((T + bm - 1) / bm) * (double)((N + bn - 1) / bn); };
    auto stage_us = [&](double wgs, double slots, double t0, double t1) {
        const double rounds = wgs <= slots ? 1.0 : (double)(int64_t)((wgs + slots - 1.0) / slots);
        return rounds * (t0 + t1 * wgs / (rounds * slots));
    };
    // W from HBM, which takes a workgroup on every compute unit (48 tokens, 4096 -> 4096: 128, 256 and 384 workgroups 19.7,
    // 17.5 and 20.8 us)
    const double stream_us = (double)Kd * N * 2 / 4.5e6;
    const int64_t all256 = (T + kGemmTileRows - 1) / kGemmTileRows;
    GemmPlan best{0, 1, (int)all256};
    double best_us = nk * stage_us(tiles_of(256, 256), kCus, 0.92, 0.78);
    for (int bm = 64; bm <= 128; bm += 64) {
        const double tiles = tiles_of(bm, GS_BN), t1 = bm == 64 ? 0.24 : 0.62;
        for (int z = 1; z <= 16; ++z) {
            if (tiles * z > 4.0 * kCus || (z > 1 && (nk < 4.0 * z || (double)z * T * N * 4 > kMaxSplitBytes))) break;
            const double steps = (double)(int64_t)((nk + z - 1.0) / z);
            double us = steps * stage_us(tiles * z, 2.0 * kCus, 0.38, t1);
            const double stream = stream_us * (tiles * z < kCus ? kCus / (tiles * z) : 1.0);
            if (us < stream) us = stream;
            if (z > 1) us += 4.0 + 0.2 * z + (double)z * T * N * 8 / 5.0e6;
            if (us < best_us) { best_us = us; best = GemmPlan{bm, z, 0}; }
        }
        // whole rounds of 256 x 256 tiles, the row tiles left over in small tiles (a launch more: 3 us)
        const int64_t cols256 = (N + 255) / 256, rounds = (int64_t)(tiles_of(256, 256) / kCus);
        const int64_t big = rounds * (int64_t)kCus / cols256;
        if (rounds < 1 || rounds > 8 || big < 1 || big >= all256) continue;
        const double rest = (double)(all256 - big) * (kGemmTileRows / bm) * (double)((N + GS_BN - 1) / GS_BN);
        if (rest > 4.0 * kCus) continue;
        const double us = 3.0 + nk * (stage_us((double)(big * cols256), kCus, 0.92, 0.78) + stage_us(rest, 2.0 * kCus, 0.38, t1));
        if (us < 0.97 * best_us) { best_us = us; best = GemmPlan{bm, 1, (int)big}; }
    }
    // 256 x 256 tiles with the contraction split
    const double tiles = tiles_of(256, 256), w_bytes = (double)Kd * N * 2, bound = best.bm == 0 ? 1.0 : s.w_cached ? 0.93 : 1.12;
    const double ext_us = all256 >= 8 || s.max_ext <= 6 ? 0.0 : (s.max_ext - 6) * (s.w_rows_contract ? 2.5 : 1.0);
    const bool whole_lines = (s.w_rows_contract ? N : Kd) % 64 == 0;
    const double lost_us = ext_us + (s.short_shrink && product_in_two_launches(best, T, N) && best.n_split >= 3 && whole_lines ? 12.0 : 0.0);
    GemmPlan split{0, 1, (int)all256};
    double split_us = bound * best_us;
    for (int z = 2; z <= (w_bytes >= 64e6 ? 6 : 4); ++z) {
        if (tiles * z > kCus || nk < 8.0 * z || (double)z * T * N * 4 > big_split_bytes) break;
        if (tiles * z < 0.75 * kCus) continue;
        const double steps = std::max((double)(int64_t)((nk + z) / z), (double)s.max_ext);
        const double us = lost_us + steps * (0.92 + 0.68 * tiles * z / kCus) + 4.0 + 0.2 * z + (double)z * T * N * 8 / 7.5e6;
        if (us < split_us) { split_us = us; split.n_split = z; }
    }
    if (T > 64 && split.n_split > 1 && best.big_tiles * best.bm == 0 && (w_bytes >= 80e6 || (double)N >= 0.98 * 256.0 * (double)((N + 255) / 256))) return split;
    return best;
}

}  // namespace plora
