// Shrink and dH of short batches (see skinny_bf16.hip for the others), as a routine of one workgroup: the preparation kernel
// runs it beside its own work, a kernel of skinny_bf16.hip for the projections of a grouped call.
//
// One workgroup (4 waves) per (slice of 16 tokens, share of the contraction).  The waves take chunks of 64 contraction elements
// in turn, operands straight from memory into registers (no barrier until the waves' sums meet in LDS), so that a chunk's loads
// are all in flight at once.  A_k is read as it lies in memory, [C][r]: 32 rows of it are one piece of memory, which goes through
// the wave's own LDS and is read back transposed; nothing has to be packed first, and nothing of the description but its words
// is needed, so the product does not wait for a preparation launch.
// With more than one share per slice the partial sums go through memory and the last workgroup to arrive at the slice -
// whichever it is - adds all of them in the order of the shares and writes the outputs; no workgroup waits for another.
// Arrival: every workgroup of a slice has a flag.  It stores the launch's own 64-bit number there behind its partial sums and
// then looks at all flags of the slice: who finds the number in all of them comes last (the last store is seen by its own
// workgroup at least; should two see it, both write the same values).  The flags are put back to zero, and what the memory held
// before the launch does not matter: no launch has cleared it.
// Bound by the start of the kernel, one trip to the description, one to the operands, one to the flags.
#pragma once
#include "plora_internal.h"

namespace plora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 sh_bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 sh_bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float sh_f32x4;

#define SH_LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

__device__ inline uint16_t bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ROWS token rows from t0 on, of which the first nt exist; tile [ROWS][r16] in LDS, 256 threads.
template <int ROWS>
__device__ inline void write_outputs(const SegInfo &g, float mult, int mode, const float *tile, int r16, int t0, int nt, const SkinnyOut &out)
{
    constexpr int TPR = 256 / ROWS;                   // threads per row
    const int hi = threadIdx.x / TPR, lo = threadIdx.x % TPR, r = g.r;
    if (out.hf && hi < nt) {
        float *dst = out.hf + g.h_off + (int64_t)(t0 + hi) * r;
        const float m = mode == 0 ? 1.f : mult;
        for (int j = lo; j < r; j += TPR) dst[j] = m * tile[hi * r16 + j];
    }
    if (out.hb && hi < nt) {
        uint4 *dst = reinterpret_cast<uint4 *>(out.hb + g.hb_off + (int64_t)(t0 + hi) * g.rp);
        for (int v = lo; v < g.rp / 8; v += TPR) {
            union { uint4 q; uint16_t h[8]; } u;
#pragma unroll
            for (int i = 0; i < 8; ++i) { const int j = v * 8 + i; u.h[i] = j < r ? bf16_rne(mult * tile[hi * r16 + j]) : (uint16_t)0; }
            dst[v] = u.q;
        }
    }
    if (out.zt) {
        const float zm = out.zt_scaled ? mult : 1.f;
        const int tt = (threadIdx.x % (ROWS / 8)) * 8;                       // 8 tokens per thread
        uint16_t *dst = out.zt + g.zt_off + t0 + tt;
        for (int j = threadIdx.x / (ROWS / 8); j < r16; j += 256 / (ROWS / 8)) {
            union { uint4 q; uint16_t h[8]; } u;
#pragma unroll
            for (int i = 0; i < 8; ++i) u.h[i] = (j < r && tt + i < nt) ? bf16_rne(zm * tile[(tt + i) * r16 + j]) : (uint16_t)0;
            *reinterpret_cast<uint4 *>(dst + (int64_t)j * g.lp) = u.q;
        }
    }
}

// Partial sums that a workgroup of another XCD reads within the launch go past the L2 (agent scope, one access at a time): a
// store is at the memory side once the wave's counter is back at zero, and the arrival is announced behind that.  A release
// and an acquire of the whole L2 instead take 0.4 us each, one after the other on an XCD (32 slices x 16 shares, 28 us against 13).
__device__ inline void store_agent(sh_f32x4 *p, sh_f32x4 v)
{
    typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
    const u64x2 q = __builtin_bit_cast(u64x2, v);
    unsigned long long *d = reinterpret_cast<unsigned long long *>(p);
    __hip_atomic_store(d, q[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(d + 1, q[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline sh_f32x4 load_agent(const sh_f32x4 *p)
{
    typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
    const unsigned long long *s = reinterpret_cast<const unsigned long long *>(p);
    u64x2 q;
    q[0] = __hip_atomic_load(s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q[1] = __hip_atomic_load(s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(sh_f32x4, q);
}
__device__ inline void wait_memory()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0): loads and stores of this wave
    asm volatile("" ::: "memory");
}

constexpr int SH_NW = 4;                              // waves per workgroup
constexpr int SH_BK = 64;                             // contraction elements per chunk
__host__ __device__ inline size_t short_lds_bytes(int r16) { return (size_t)SH_NW * 64 * r16 + 16; }

// g, scale: the slice's segment; t0: its first token inside the segment; unit: index of the slice; small: B_k (mode 1: [r][C]),
// A_k as it is (mode 0, natural: [C][r]) or packed (mode 0: [r16][C]).
// PARTS: the sums of every share go to `part` and are added by a later launch.
// (Inlining is left to the compiler: forced, k_prep_short<1> took 128 registers instead of 104 and 3 to 6 % longer, 926 tokens, 992 -> 17408 beside
// a caller's product 78.3 us for a step and 77.3.)
template <int NB, bool PARTS = false>
__device__ inline void skinny_short(const ShortJob &job, const SegInfo &g, float scale, int t0, int unit, int n_units, int split,
                                    const uint16_t *small, bool natural, char *lds)
{
    float *red = reinterpret_cast<float *>(lds);                      // [SH_NW][16][r16]
    if (t0 >= g.lp) return;
    const int nt = g.row1 - g.row0 - t0;
    if (nt <= 0) {                                                    // padding tokens alone: the transposed copy has zeros there
        if (split == 0 && job.out.zt) write_outputs<16>(g, scale, job.mode, red, g.r16, t0, 0, job.out);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lm = lane & 15, kg = lane >> 4;
    const int C = job.C, r = g.r, r16 = g.r16, nb = r16 / 16;
    const uint16_t *xrow = job.S + (int64_t)(g.row0 + t0 + (lm < nt ? lm : nt - 1)) * C;    // rows past the end only feed sums that are not stored
    sh_f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = sh_f32x4{0.f, 0.f, 0.f, 0.f};
    const int n_chunks = (C + SH_BK - 1) / SH_BK, c_lo = split * job.per;
    const int c_hi = c_lo + job.per < n_chunks ? c_lo + job.per : n_chunks;
    const sh_bf16x8 none = {};
    char *slab = lds + wave * (64 * r16);                             // the wave's 32 rows of A_k
    // H: half chunks (32 elements) of a wave in flight together (PARTS: beside a product that leaves twice the registers)
    constexpr int H = (NB <= 1 ? 8 : NB <= 2 ? 4 : NB <= 4 ? 2 : 1) * (PARTS && NB > 1 ? 2 : 1);
    const int n_half = c_hi > c_lo + wave ? ((c_hi - c_lo - wave - 1) / SH_NW + 1) * 2 : 0;     // of this wave
    for (int h0 = 0; h0 < n_half; h0 += H) {
        sh_bf16x8 xf[H], bf[H][NB];
#pragma unroll
        for (int u = 0; u < H; ++u) {
            if (h0 + u >= n_half) break;
            const int k0 = (c_lo + wave + (h0 + u) / 2 * SH_NW) * SH_BK + (h0 + u) % 2 * 32, k = k0 + kg * 8;
            const bool whole = k0 + 32 <= C, ok = whole || k < C;     // elements past the end are zero in both operands
            xf[u] = *reinterpret_cast<const sh_bf16x8 *>(xrow + (ok ? k : 0));
            if (!ok) xf[u] = none;
            if (natural) {
                const int rows = whole ? 32 : C - k0, pieces = rows > 0 ? rows * r / 8 : 0;
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b < nb) {
                        const int p = b * 64 + lane;
                        const bool in = p < pieces;
                        bf[u][b] = *reinterpret_cast<const sh_bf16x8 *>(small + (in ? (int64_t)k0 * r + p * 8 : 0));
                        if (!in) bf[u][b] = none;
                    }
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b < nb) {
                        const int j = b * 16 + lm;                    // rows past the rank only feed columns that are not stored
                        bf[u][b] = *reinterpret_cast<const sh_bf16x8 *>(small + (int64_t)(j < r ? j : 0) * C + (ok ? k : 0));
                        if (!ok) bf[u][b] = none;
                    }
            }
        }
#pragma unroll
        for (int u = 0; u < H; ++u) {
            if (h0 + u >= n_half) break;
            if (natural) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b < nb && b * 64 + lane < 4 * r) *reinterpret_cast<sh_bf16x8 *>(slab + (b * 64 + lane) * 16) = bf[u][b];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (b >= nb) continue;
                    if ((r & 3) == 0) {
                        // transposing read: the 16 lanes of a group fetch a 4(k) x 16 block; lane i then holds column i
                        const char *q = slab + ((kg * 8 + (lm >> 2)) * r + b * 16 + (lm & 3) * 4) * 2;
                        const sh_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(SH_LDS_PTR(sh_bf16x4, q));
                        const sh_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(SH_LDS_PTR(sh_bf16x4, q + 8 * r));
                        bf[u][b] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    } else {
                        union { sh_bf16x8 v; uint16_t h[8]; } f;
#pragma unroll
                        for (int i = 0; i < 8; ++i) f.h[i] = reinterpret_cast<const uint16_t *>(slab)[(kg * 8 + i) * r + b * 16 + lm];
                        bf[u][b] = f.v;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (b < nb) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[u], bf[u][b], acc[b], 0, 0, 0);
        }
    }
    // sums of the waves, in wave order: element e of [16][r16].  (A wave's part of `red` is where its own slab was.)
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (b < nb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) red[(wave * 16 + kg * 4 + i) * r16 + b * 16 + lm] = acc[b][i];
        }
    __syncthreads();
    const int n_vec = 4 * r16;
    sh_f32x4 *red4 = reinterpret_cast<sh_f32x4 *>(red);
    const int64_t stride = (int64_t)n_units * 4 * job.max_r16;        // of the partial sums of one share
    sh_f32x4 *part4 = reinterpret_cast<sh_f32x4 *>(job.part) + (int64_t)unit * 4 * job.max_r16;
    for (int e = threadIdx.x; e < n_vec; e += 64 * SH_NW) {
        sh_f32x4 v = red4[e];
#pragma unroll
        for (int w = 1; w < SH_NW; ++w) v += red4[w * n_vec + e];
        if constexpr (PARTS) part4[split * stride + e] = v;
        else if (job.n_split > 1) store_agent(part4 + split * stride + e, v);
        else red4[e] = v;
    }
    if constexpr (PARTS) return;
    if (job.n_split > 1) {
        wait_memory();
        __syncthreads();
        uint32_t *last = reinterpret_cast<uint32_t *>(red4 + SH_NW * n_vec);
        unsigned long long *flag = job.flags + (int64_t)unit * kShortMaxSplits;
        if (wave == 0) {
            if (lane == 0) __hip_atomic_store(flag + split, job.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_memory();
            bool here = true;
            if (lane < job.n_split) here = __hip_atomic_load(flag + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == job.number;
            const bool all = __ballot(here) == ~0ull;
            if (all && lane < job.n_split) __hip_atomic_store(flag + lane, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) *last = all ? 1u : 0u;
        }
        __syncthreads();
        if (*last == 0u) return;
        for (int e = threadIdx.x; e < n_vec; e += 64 * SH_NW) {
            sh_f32x4 sum = load_agent(part4 + e);
            for (int s0 = 1; s0 < job.n_split; s0 += 5) {
                sh_f32x4 v[5];
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    if (s0 + i < job.n_split) v[i] = load_agent(part4 + (s0 + i) * stride + e);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    if (s0 + i < job.n_split) sum += v[i];
            }
            red4[e] = sum;
        }
    }
    __syncthreads();
    write_outputs<16>(g, scale, job.mode, red, r16, t0, nt < 16 ? nt : 16, job.out);
}

}  // namespace plora
