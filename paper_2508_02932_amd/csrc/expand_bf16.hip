// Stand-alone low-rank update of the packed multi-LoRA layer on bf16 inputs (gfx950), for callers that
// compute the base product themselves:
//   forward   y_t  += scale_k (x_t A_k) B_k      (section 2.4: the low-rank half of the layer)
//   backward  dx_t += g_t A_k^T                  (appendix C.2, case 4: its low-rank half)
// C[T][N] is read, updated in fp32 and written back once (rounded to nearest even), so the kernel is
// bound by HBM: 2 x 2 bytes per element of C.  The two small operands come as the other kernels of the
// library already keep them: the bf16 low-rank factor [len][rp] of each segment (scale_k h, or g) and
// the padded, transposed small matrix [N][rp] (B_k^T, or A_k), both with zeros beyond the rank, so a
// lane fetches its MFMA operands as 16 contiguous bytes straight from L2 and the rank is never tiled
// (appendix C.2).  Only the C tile goes through LDS: it comes in by direct loads in whole 128-byte
// row pieces (512 bytes per row and workgroup), is read and rewritten there in the MFMA accumulator layout, and leaves in whole row
// pieces again.  Every wave owns 64 columns of the tile, so no workgroup barrier is needed.
// 16384 tokens, 8 adapters of rank 8 to 128: y with 14336 columns 225 -> 204 us (4.6 TB/s), dx with 4096 columns 72 -> 62 us,
// against tiles of 128 tokens x 128 columns with the token blocks fastest (half as many bytes side by side in a row of C,
// and 20 % more operand traffic from L2); a copy of y takes 186 us.
#include "plora_internal.h"

namespace plora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int EX_COLS = 256;                       // columns of C per workgroup (512 bytes per row), 64 per wave
constexpr int EX_ROWS = 64;                        // token rows per workgroup
constexpr int EX_NW = EX_COLS / 64;
constexpr int EX_LDS = EX_ROWS * EX_COLS * 2;      // 32 KB, 8 KB per wave

__device__ inline uint32_t ex_pack_bf16x2(float lo, float hi)
{
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}

// One workgroup per (half of a token block of one segment, 256 columns of C), the column tiles fastest: workgroups that run
// side by side then cover whole rows of C, and with a multiple of 8 tiles an XCD keeps meeting the same columns of opT.
//   side : bf16 low-rank factor, segment s at side + hb_off, rows of rp elements
//   opT  : small matrices [N][rp], adapter k behind N * rp elements of every adapter before it
// PAST: C is larger than the last cache, so nothing of it is there when anything reads it again: it is read and written with the
// non-temporal hint, if its rows are whole lines of 128 bytes (otherwise neighbouring tiles share lines: 4096 ->
// 8200 605 -> 635 us).  Forward and backward of 16384 tokens, 4096 -> 14336, eight adapters of rank 8 to 128 808 -> 784 us, rank 32
// 760 -> 736: 5 us in this kernel, the rest in what runs after it and no longer waits for lines of C to be written back.
// part0: the first half block of the launch.  KS: 32-rank MFMA steps that the largest rank of the launch needs (1, 2 or 4).
template <int KS, bool PAST>
__global__ void __launch_bounds__(64 * EX_NW, KS == 4 ? 3 : 4) k_expand(MetaView mv, uint16_t *__restrict__ C, int N, int tiles_n, int part0,
                                                       const uint16_t *__restrict__ side, const uint16_t *__restrict__ opT,
                                                       const uint16_t *__restrict__ zero)
{
    __shared__ __attribute__((aligned(1024))) char lds[EX_LDS];
    constexpr int kHalves = kSkinnyRows / EX_ROWS;
    const int rel = blockIdx.x / tiles_n, n_tile = blockIdx.x - rel * tiles_n, part = part0 + rel;
    const BlkInfo bi = mv.blk[part / kHalves];
    const SegInfo g = bi.g;
    const int t0 = bi.t0 + (part % kHalves) * EX_ROWS;
    const int left = g.row1 - g.row0 - t0;
    if (left <= 0) return;
    const int nt = left < EX_ROWS ? left : EX_ROWS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = n_tile * EX_COLS + wave * 64;
    if (n0 >= N) return;                           // every wave works alone: no barrier below
    const int rp = g.rp;
    const int ksteps = (g.r + 31) / 32;            // 32 rank columns per MFMA; columns r .. 32 ksteps are zero on both sides
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(char, lds)) + wave * (EX_ROWS * 128);
    char *tile = lds + wave * (EX_ROWS * 128);

    // ---- C tile -> LDS.  A load instruction moves 8 rows x 128 bytes: lane -> (row 8q + lane/8, slot lane%8); slot c'
    // of row u holds the 16-byte chunk c' ^ (u & 7), so that the rows read together below spread over the banks.
    uint16_t *Crow0 = C + (int64_t)(g.row0 + t0) * N + n0;
    const int lrow = lane >> 3, slot = lane & 7;
    const int ccol = (slot ^ lrow) * 8;            // (8q + lane/8) & 7 = lane/8
    const bool cok = n0 + ccol < N;
#pragma unroll
    for (int j = 0; j < EX_ROWS / 8; ++j) {
        const int u = j * 8 + lrow;
        const void *src = (u < nt && cok) ? static_cast<const void *>(Crow0 + (int64_t)u * N + ccol) : static_cast<const void *>(zero);
        if constexpr (PAST) asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "s"(lds_base + j * 1024));
        else asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_base + j * 1024));
    }

    // ---- low-rank operands straight from memory (they sit in L2).  MFMA 16x16x32: the first operand's rows are columns n
    // of C, the second operand's columns are token rows, so a lane ends up with 4 consecutive n of one token.
    const int lm = lane & 15, kg = lane >> 4;
    const uint16_t *op = opT + bi.rp_off * (int64_t)N;                    // this adapter's [N][rp]
    bf16x8 sf[4][KS], bfr[2][KS];
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
        int u = tb * 16 + lm;
        u = u < nt ? u : nt - 1;                                          // clamped rows are never stored
        const uint16_t *p = side + g.hb_off + (int64_t)(t0 + u) * rp + kg * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            if (ks < ksteps) sf[tb][ks] = *reinterpret_cast<const bf16x8 *>(p + ks * 32);
    }
    auto load_block = [&](int b, bf16x8 *dst) {                           // small-matrix rows of column block b
        int n = n0 + b * 16 + lm;
        n = n < N ? n : N - 1;                                            // clamped columns are never stored
        const uint16_t *p = op + (int64_t)n * rp + kg * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            if (ks < ksteps) dst[ks] = *reinterpret_cast<const bf16x8 *>(p + ks * 32);
    };
    load_block(0, bfr[0]);
    load_block(1, bfr[1]);

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                    // this wave's tile is in LDS
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            // accumulator of (token 16tb + lm, columns 16b + 4kg .. +3): 8 bytes of the tile
            const int u = tb * 16 + lm;
            const int chunk = 2 * b + (kg >> 1);
            char *cell = tile + u * 128 + ((chunk ^ (u & 7)) * 16) + (kg & 1) * 8;
            const u32x2 old = *LDS_PTR(const u32x2, cell);
            f32x4 v;
            v[0] = __uint_as_float(old.x << 16); v[1] = __uint_as_float(old.x & 0xffff0000u);
            v[2] = __uint_as_float(old.y << 16); v[3] = __uint_as_float(old.y & 0xffff0000u);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                if (ks < ksteps) v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[b & 1][ks], sf[tb][ks], v, 0, 0, 0);
            u32x2 nu;
            nu.x = ex_pack_bf16x2(v[0], v[1]);
            nu.y = ex_pack_bf16x2(v[2], v[3]);
            *LDS_PTR(u32x2, cell) = nu;
        }
        if (b + 2 < 4) load_block(b + 2, bfr[b & 1]);                     // flies while the other block is multiplied
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                  // the wave's own writes, before it reads them back
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < EX_ROWS / 8; ++j) {
        const int u = j * 8 + lrow;
        const u32x4 v = *LDS_PTR(const u32x4, tile + j * 1024 + lane * 16);
        u32x4 *dst = reinterpret_cast<u32x4 *>(Crow0 + (int64_t)u * N + ccol);
        if (u < nt && cok) {
            if constexpr (PAST) __builtin_nontemporal_store(v, dst);
            else *dst = v;
        }
    }
}

hipError_t launch_expand_bf16(const MetaView &mv, const MetaHeader &h, void *C, int64_t N, const void *side, const void *opT,
                              const void *zero, hipStream_t st)
{
    if (h.n_blocks == 0) return hipSuccess;
    const int64_t tiles_n = (N + EX_COLS - 1) / EX_COLS;
    const bool past = h.T * N * 2 > kLastCacheBytes && rows_of_whole_lines(C, N);
    // A launch has fewer than 2^32 threads, which one-row segments of a very wide C exceed (1024 of them, 2^22 columns: 2^33):
    // as many launches as it takes, whole half blocks in each.
    const int64_t parts = (int64_t)h.n_blocks * (kSkinnyRows / EX_ROWS), per_launch = ((((int64_t)1 << 32) - 1) / (64 * EX_NW)) / tiles_n;
    for (int64_t p0 = 0; p0 < parts; p0 += per_launch) {
        const unsigned n_wg = (unsigned)((parts - p0 < per_launch ? parts - p0 : per_launch) * tiles_n);
#define PL_EX_(KS_, PAST_) hipLaunchKernelGGL((k_expand<KS_, PAST_>), dim3(n_wg), dim3(64 * EX_NW), 0, st, mv, static_cast<uint16_t *>(C), \
                                      (int)N, (int)tiles_n, (int)p0, static_cast<const uint16_t *>(side), static_cast<const uint16_t *>(opT), \
                                      static_cast<const uint16_t *>(zero))
#define PL_EX(KS_) do { if (past) PL_EX_(KS_, true); else PL_EX_(KS_, false); } while (0)
        if (h.max_r16 <= 32) PL_EX(1);
        else if (h.max_r16 <= 64) PL_EX(2);
        else PL_EX(4);
#undef PL_EX
#undef PL_EX_
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace plora
