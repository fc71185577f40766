// Small helper kernels of libplora: derivation of the metadata tables from the compact description
// (which travels as a kernel argument), zero page, packing of the adapter matrices into
// MFMA-friendly bf16 buffers, transposed copy of a saved activation.
#include "plora_internal.h"
#include "nf4_expand.h"
#include "prep.h"
#include "skinny_short.h"
#include "f32_tiles.h"

#include <atomic>
#include <cstring>
#include <mutex>
#include <random>

namespace plora {

// ---- per-device state ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
static std::mutex g_dev_mu;
static int g_cu[kMaxDevices];
static bool g_lds_ok[kMaxDevices][kLdsSlots];

int device_cu_count(hipError_t *err)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) { *err = e != hipSuccess ? e : hipErrorInvalidDevice; return 0; }
    std::lock_guard<std::mutex> lock(g_dev_mu);
    if (g_cu[dev] == 0) {
        int v = 0;
        e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess || v < 1) { *err = e != hipSuccess ? e : hipErrorInvalidDevice; return 0; }
        g_cu[dev] = v;
    }
    *err = hipSuccess;
    return g_cu[dev];
}

hipError_t allow_full_lds(const void *kernel, int slot)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices || slot < 0 || slot >= kLdsSlots) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(g_dev_mu);
    if (!g_lds_ok[dev][slot]) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        g_lds_ok[dev][slot] = true;
    }
    return hipSuccess;
}

// ---- chunked upload of a compact description too long for one kernel argument ----------------------
__global__ void __launch_bounds__(256) k_upload(DescChunk c, uint32_t *dst, int n_words)
{
    for (int i = threadIdx.x; i < n_words; i += 256) dst[i] = c.w[i];
}

static hipError_t upload_words(uint32_t *dst_dev, const uint32_t *src_host, int n_words, hipStream_t st)
{
    for (int w0 = 0; w0 < n_words; w0 += kChunkWords) {
        DescChunk c;
        const int nw = n_words - w0 < kChunkWords ? n_words - w0 : kChunkWords;
        std::memcpy(c.w, src_host + w0, (size_t)nw * 4);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, st, c, dst_dev + w0, nw);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- the preparation kernels (device code in prep.h) --------------------------------------------------
__global__ void __launch_bounds__(256) k_prep_arg(DescChunk c, PrepArgs pa)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    prep_body(DescReader<WordsInArg>{WordsInArg{c.w}}, pa, blockIdx.x, prep_lds);
}

// The workgroups behind the preparation's expand an NF4 weight: 58.7 M weights take 27 us, the preparation of a small batch 9 us
// of mostly latency, and neither waits for the other.
template <bool BF16>
__global__ void __launch_bounds__(256) k_prep_nf4(DescChunk c, PrepArgs pa, Nf4Job w, int n_prep)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    if ((int)blockIdx.x < n_prep) prep_body(DescReader<WordsInArg>{WordsInArg{c.w}}, pa, blockIdx.x, prep_lds);
    else nf4_expand<BF16>(w.codes, w.absmax, w.out, w.n_elems / 8, blockIdx.x - n_prep, gridDim.x - n_prep, reinterpret_cast<float *>(prep_lds));
}

// Short products in the same launch (skinny_short.h): they read the description's words and the call's own operands alone, so
// shrink and dH run beside the preparation instead of behind it.  Workgroups: the preparation's, then the products'.
// Preparation, product and finishing launch before, and this launch now, us: 512 tokens, 4096 columns, rank 16 17 and 10, 14336
// columns 21 and 14; 48 tokens of eight adapters, 4096 columns 20 and 14; 1531 tokens, 1000 columns, rank 100 22 and 18.
struct PrepShort { ShortJob j[kPrepShort]; };
template <int NB>
__global__ void __launch_bounds__(256, NB == 8 ? 3 : 4) k_prep_short(DescChunk c, PrepArgs pa, PrepShort sj, int n_jobs, int n_units, int n_prep)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    const DescReader<WordsInArg> in{WordsInArg{c.w}};
    int wg = blockIdx.x;
    if (wg < n_prep) { prep_body(in, pa, wg, prep_lds); return; }
    wg -= n_prep;
    const ShortJob job = sj.j[n_jobs > 1 && wg >= sj.j[1].wg0 ? 1 : 0];
    wg -= job.wg0;
    const int split = wg / n_units, unit = wg - split * n_units;
    int t_block;
    float scale;
    const SegInfo g = segment_of_block(in, unit / kShortSlices, t_block, scale);
    const int t0 = t_block + unit % kShortSlices * 16;
    if (t0 >= g.lp) return;
    skinny_short<NB>(job, g, scale, t0, unit, n_units, split, static_cast<const uint16_t *>(in.ad_ptr(g.adapter, job.mode == 0 ? 0 : 1)),
                     job.mode == 0, prep_lds);
}

// The fp32 path: its low-rank products of any size (16 tokens x 16 ranks per workgroup; they are a small part of a call).
struct PrepF32 { F32LowRank j[kPrepShort]; };
__global__ void __launch_bounds__(256, 4) k_prep_f32(DescChunk c, PrepArgs pa, PrepF32 fj, int n_units, int tiles_j, int n_prep)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    const DescReader<WordsInArg> in{WordsInArg{c.w}};
    int wg = blockIdx.x;
    if (wg < n_prep) { prep_body(in, pa, wg, prep_lds); return; }
    wg -= n_prep;
    const int per_job = n_units * tiles_j, which = wg / per_job;
    wg -= which * per_job;
    const F32LowRank job = fj.j[which];
    const int unit = wg / tiles_j, j0 = (wg - unit * tiles_j) * 16;
    int t_block;
    float scale;
    const SegInfo g = segment_of_block(in, unit / kShortSlices, t_block, scale);
    if (j0 >= g.r) return;
    f32_lowrank_tile(job, g, scale, static_cast<const float *>(in.ad_ptr(g.adapter, job.mode == 0 ? 0 : 1)), t_block + unit % kShortSlices * 16, j0,
                     reinterpret_cast<double *>(prep_lds));
}

__global__ void __launch_bounds__(256) k_prep_batch(PrepBatch c)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    int i = 0;
    for (int q = 1; q < kMaxGroup; ++q)
        if (q < c.n && (int)blockIdx.x >= c.a[q].block0) i = q;
    prep_body(DescReader<WordsInArg>{WordsInArg{c.w + c.a[i].word0}}, c.a[i], (int)blockIdx.x - c.a[i].block0, prep_lds);
}

__global__ void __launch_bounds__(256) k_prep_mem(const uint32_t *desc, PrepArgs pa)
{
    extern __shared__ __attribute__((aligned(16))) char prep_lds[];
    prep_body(DescReader<WordsInMemory>{WordsInMemory{desc}}, pa, blockIdx.x, prep_lds);
}

unsigned long long launch_number()
{
    static std::atomic<unsigned long long> next{((unsigned long long)std::random_device{}() << 32) | 1u};
    unsigned long long v = next.fetch_add(1);
    return v ? v : next.fetch_add(1);
}

// The preparation with the short products of the call.
static hipError_t launch_prep_short(const PrepJob &j, hipStream_t st)
{
    if (j.n_brief < 1 || j.n_brief > kPrepShort || j.n_words > kChunkWords) return hipErrorInvalidValue;
    PrepArgs pa;
    int64_t n_wg;
    size_t lds;
    hipError_t e = prep_args(j, pa, n_wg, lds);
    if (e != hipSuccess) return e;
    const int n_units = j.h.n_blocks * kShortSlices;
    PrepShort sj{};
    int n_short = 0;
    for (int i = 0; i < j.n_brief; ++i) {
        sj.j[i] = short_job(j.brief[i]);
        sj.j[i].wg0 = n_short;
        n_short += n_units * sj.j[i].n_split;
    }
    if (lds < short_lds_bytes(j.h.max_r16)) lds = short_lds_bytes(j.h.max_r16);
    DescChunk c;
    std::memcpy(c.w, j.desc_host, (size_t)j.n_words * 4);
    const dim3 grid((unsigned)(n_wg + n_short));
    const int nb = j.h.max_r16 / 16;
#define PL_PS(NB_) hipLaunchKernelGGL(k_prep_short<NB_>, grid, dim3(256), lds, st, c, pa, sj, j.n_brief, n_units, (int)n_wg)
    if (nb <= 1) PL_PS(1);
    else if (nb <= 2) PL_PS(2);
    else if (nb <= 4) PL_PS(4);
    else PL_PS(8);
#undef PL_PS
    return hipGetLastError();
}

static hipError_t launch_prep_f32(const PrepJob &j, hipStream_t st)
{
    if (j.n_f32 < 1 || j.n_f32 > kPrepShort || j.n_words > kChunkWords) return hipErrorInvalidValue;
    PrepArgs pa;
    int64_t n_wg;
    size_t lds;
    hipError_t e = prep_args(j, pa, n_wg, lds);
    if (e != hipSuccess) return e;
    const int n_units = j.h.n_blocks * kShortSlices, tiles_j = j.h.max_r16 / 16;
    PrepF32 fj{};
    for (int i = 0; i < j.n_f32; ++i) fj.j[i] = j.f32[i];
    constexpr size_t need = F32_NW * 16 * 16 * sizeof(double);
    if (lds < need) lds = need;
    DescChunk c;
    std::memcpy(c.w, j.desc_host, (size_t)j.n_words * 4);
    hipLaunchKernelGGL(k_prep_f32, dim3((unsigned)(n_wg + (int64_t)n_units * tiles_j * j.n_f32)), dim3(256), lds, st, c, pa, fj, n_units, tiles_j, (int)n_wg);
    return hipGetLastError();
}

static hipError_t launch_prep_one(const PrepJob &j, hipStream_t st)
{
    if (j.n_f32 > 0) return launch_prep_f32(j, st);
    if (j.dh) return launch_prep_dh(j, st);
    if (j.n_brief > 0) return launch_prep_short(j, st);
    PrepArgs pa;
    int64_t n_wg;
    size_t lds;
    hipError_t e = prep_args(j, pa, n_wg, lds);
    if (e != hipSuccess) return e;
    if (j.n_words <= kChunkWords) {
        DescChunk c;
        std::memcpy(c.w, j.desc_host, (size_t)j.n_words * 4);
        hipLaunchKernelGGL(k_prep_arg, dim3((unsigned)n_wg), dim3(256), lds, st, c, pa);
        return hipGetLastError();
    }
    e = upload_words(j.desc_stage, j.desc_host, j.n_words, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_prep_mem, dim3((unsigned)n_wg), dim3(256), lds, st, static_cast<const uint32_t *>(j.desc_stage), pa);
    return hipGetLastError();
}

hipError_t launch_prep_nf4(const PrepJob &j, const Nf4Job &w, bool bf16, hipStream_t st)
{
    if (j.n_brief > 0 || j.n_f32 > 0 || j.dh) return hipErrorInvalidValue;
    PrepArgs pa;
    int64_t n_wg;
    size_t lds;
    hipError_t e = prep_args(j, pa, n_wg, lds);
    if (e != hipSuccess) return e;
    const int n_nf4 = nf4_workgroups(w.n_elems);
    if (n_nf4 < 1) return hipErrorInvalidDevice;
    // a launch takes its LDS from the larger part: above 20 KB the expansion would lose workgroups to it
    if (j.n_words > kChunkWords || lds > 20 * 1024) {
        e = launch_nf4_dequant(w.codes, w.absmax, w.n_elems, bf16, w.out, st);
        return e != hipSuccess ? e : launch_prep_one(j, st);
    }
    DescChunk c;
    std::memcpy(c.w, j.desc_host, (size_t)j.n_words * 4);
    const dim3 grid((unsigned)(n_wg + n_nf4));
    if (bf16) hipLaunchKernelGGL(k_prep_nf4<true>, grid, dim3(256), lds, st, c, pa, w, (int)n_wg);
    else hipLaunchKernelGGL(k_prep_nf4<false>, grid, dim3(256), lds, st, c, pa, w, (int)n_wg);
    return hipGetLastError();
}

hipError_t launch_prep(const PrepJob *jobs, int n_jobs, hipStream_t st)
{
    int words = 0;
    for (int i = 0; i < n_jobs; ++i) words += jobs[i].n_words;
    if (n_jobs == 1 || n_jobs > kMaxGroup || words > kPrepBatchWords) {
        for (int i = 0; i < n_jobs; ++i) {
            const hipError_t e = launch_prep_one(jobs[i], st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    PrepBatch c;
    c.n = n_jobs; c.pad = 0;
    int64_t blocks = 0;
    size_t lds = 0;
    for (int i = 0, w = 0; i < n_jobs; ++i) {
        int64_t n_wg;
        size_t one;
        const hipError_t e = prep_args(jobs[i], c.a[i], n_wg, one);
        if (e != hipSuccess) return e;
        c.a[i].word0 = w; c.a[i].block0 = (int32_t)blocks;
        std::memcpy(c.w + w, jobs[i].desc_host, (size_t)jobs[i].n_words * 4);
        w += jobs[i].n_words; blocks += n_wg;
        lds = one > lds ? one : lds;
    }
    hipLaunchKernelGGL(k_prep_batch, dim3((unsigned)blocks), dim3(256), lds, st, c);
    return hipGetLastError();
}

}  // namespace plora
